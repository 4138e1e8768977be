// Group-aligned sliced first output projection with artifact restore-and-replace
// (eq:offonline, eq:factorization, Alg. 2: z_online = W_{a,G} O_G + W_{a,L} O_{L,A};
// z = z_online + z_off on unprotected rows, z = z_online on protected rows).
//
// Two bf16 MFMA GEMM passes per projection group pg, both on the caller's stream:
//   pass G: every row, K = the Global heads of pg's groups; the epilogue adds
//           z_off[r] on unprotected rows and nothing on protected rows, so
//           z_off is never read for protected rows (the replace);
//   pass L: rows a of the protected set, K = the Local heads of pg's groups;
//           the result is added to the pass-G value in z[prot_rows[a]].
// Pass G's epilogue loads the values it adds a 32-row block at a time, before the
// block's first store, so that their latencies overlap.
// Each head's weight rows are a d_c-row block of w_o[pg]; a K tile of 64 never
// straddles two heads, so the B operand is gathered per tile by head.  The MFMAs
// compute the transposed tile (W^T O^T), so that each lane holds one output row
// and runs of 4 consecutive channels: the epilogue reads z_off and writes z 8 and
// 16 bytes at a time.
#include "oproj.h"

#include <algorithm>
#include <type_traits>

namespace mla {

// Tile shapes: BM rows x BN channels per workgroup of WM x WN waves (wave tiles
// of multiples of 32), K in steps of 64.
constexpr int OP_BK = 64;
constexpr int OP_ALD = OP_BK + 8;     // padded A row (bf16): 144 B, conflict-free 16-byte row reads

template <int BM, int BN, int WM, int WN>   // pass G
// at most 128 registers per wave, so that two workgroups of 8 waves share a CU
__global__ __launch_bounds__(WM * WN * 64) __attribute__((amdgpu_waves_per_eu(4)))
void oproj_kernel(OprojArgs a, int m_tiles, int n_tiles) {
  constexpr int NT = WM * WN * 64;
  // padded B row: 2*BLD = 64 mod 256 bytes, so the four k-rows that each half-wave
  // of a transposing read touches land on disjoint 16-bank groups (all 64 banks)
  constexpr int OP_BLD = BN + 32;
  constexpr int TM = BM / WM, TN = BN / WN;    // wave tile
  constexpr int MI = TM / 32, NI = TN / 32;     // 32x32 MFMA blocks per wave
  constexpr int A_CH = BM * OP_BK / 8 / NT;     // 16-byte chunks per thread and K step
  constexpr int B_CH = OP_BK * BN / 8 / NT;
  static_assert(TM % 32 == 0 && TN % 32 == 0 && A_CH >= 1 && B_CH >= 1, "tile shape");
  static_assert(((2 * OP_BLD) % 256) == 64, "B row padding");
  constexpr int OP_BM = BM, OP_BN = BN;
  // one LDS buffer per operand: the next K step waits in registers, and two
  // workgroups fit a CU, one's epilogue running beside the other's K loop
  __shared__ __attribute__((aligned(16))) uint16_t As[OP_BM * OP_ALD];
  __shared__ __attribute__((aligned(16))) uint16_t Bs[OP_BK * OP_BLD];
  __shared__ int row_flag[OP_BM];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hpg = a.n_heads / a.n_groups;
  const int gpp = a.n_groups / a.n_pg;              // output groups per projection group
  const int cw = a.d_model / a.n_pg;                // channels per projection group
  const int heads_pp = a.n_heads / a.n_pg;
  const int DC = a.d_latent;

  // XCD-aware tile order: workgroups go to the 8 XCDs round-robin by id, so XCD x
  // takes the contiguous tile range [x*per, (x+1)*per); the n_tiles column tiles
  // of one row block are consecutive and share that row block in the XCD's L2
  const int total = n_tiles * m_tiles * a.n_pg;
  const int per = (total + 7) / 8;
  int bid = (int)(blockIdx.x % 8) * per + (int)(blockIdx.x / 8);
  if (bid >= total) return;
  const int nt = bid % n_tiles;
  bid /= n_tiles;
  const int mt = bid % m_tiles;
  const int pg = bid / m_tiles;
  const int m0 = mt * OP_BM, n0 = nt * OP_BN;

  // protected rows in use: the host count, or the device count clamped to the capacity
  int n_prot = a.n_prot;
  if (a.n_prot_dev != nullptr) {
    const int d = *a.n_prot_dev;
    n_prot = d < 0 ? 0 : (d < a.n_prot ? d : a.n_prot);
  }
  const int64_t M = a.n_rows;
  const int K = gpp * DC;   // one d_c-wide K block per Global head
  const uint16_t* A = (const uint16_t*)a.o_glob;
  const int64_t lda = (int64_t)a.n_groups * DC;
  const int64_t acol = (int64_t)pg * gpp * DC;
  const uint16_t* W = (const uint16_t*)a.w_o + (int64_t)pg * heads_pp * DC * cw;

  {
    // the tile's rows are [m0, m0 + BM): the protected ones are the run of the
    // sorted list between two lower bounds, found once per workgroup
    __shared__ int run[2];
    if (tid < 2) {
      const int64_t key = tid == 0 ? (int64_t)m0 : (int64_t)m0 + OP_BM;
      int lo = 0, hi = n_prot;
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if ((int64_t)a.prot_rows[mid] < key) lo = mid + 1; else hi = mid;
      }
      run[tid] = lo;
    }
    for (int i = tid; i < OP_BM; i += NT) row_flag[i] = 0;
    __syncthreads();
    for (int k = run[0] + tid; k < run[1]; k += NT) {
      const int64_t r = (int64_t)a.prot_rows[k] - m0;
      if (r >= 0 && r < OP_BM) row_flag[r] = 1;   // in range for any list, sorted or not
    }
  }

  // weight row of K index k (k is a multiple of 32 inside one head block)
  auto w_row = [&](int k) -> int64_t {
    const int kb = k / DC, d = k - kb * DC;
    const int hl = kb * hpg + a.glob_head[pg * gpp + kb];   // head inside the projection group
    return (int64_t)hl * DC + d;
  };

  u32x4 ra[A_CH], rb[B_CH];
  auto load_tiles = [&](int k0) {
#pragma unroll
    for (int i = 0; i < A_CH; ++i) {
      const int c = tid + NT * i;
      const int r = c / (OP_BK / 8), cc = c % (OP_BK / 8);
      int64_t m = m0 + r;
      if (m >= M) m = M - 1;
      ra[i] = *(const u32x4*)(A + m * lda + acol + k0 + cc * 8);
    }
    const int64_t wr = w_row(k0);
#pragma unroll
    for (int i = 0; i < B_CH; ++i) {
      const int c = tid + NT * i;
      const int kr = c / (OP_BN / 8), cc = c % (OP_BN / 8);
      const int n = n0 + cc * 8;
      if (n < cw)
        rb[i] = *(const u32x4*)(W + (wr + kr) * cw + n);
      else
        rb[i] = u32x4{0u, 0u, 0u, 0u};
    }
  };
  auto store_tiles = [&]() {
#pragma unroll
    for (int i = 0; i < A_CH; ++i) {
      const int c = tid + NT * i;
      *(u32x4*)(&As[(c / (OP_BK / 8)) * OP_ALD + (c % (OP_BK / 8)) * 8]) = ra[i];
    }
#pragma unroll
    for (int i = 0; i < B_CH; ++i) {
      const int c = tid + NT * i;
      *(u32x4*)(&Bs[(c / (OP_BN / 8)) * OP_BLD + (c % (OP_BN / 8)) * 8]) = rb[i];
    }
  };

  f32x16 acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  const int wm = wave / WN, wn = wave % WN;
  const int half = lane >> 5, l32 = lane & 31;
  const int q = lane >> 4, j16 = lane & 15;

  load_tiles(0);
  store_tiles();
  __syncthreads();
  const int nk = K / OP_BK;
  for (int it = 0; it < nk; ++it) {
    if (it + 1 < nk) load_tiles((it + 1) * OP_BK);
#pragma unroll
    for (int ks = 0; ks < OP_BK / 16; ++ks) {
      bf16x8 af[MI], bfr[NI];
#pragma unroll
      for (int mi = 0; mi < MI; ++mi)
        af[mi] = *(const bf16x8*)(&As[(wm * TM + mi * 32 + l32) * OP_ALD + ks * 16 + half * 8]);
#pragma unroll
      for (int ni = 0; ni < NI; ++ni) {
        // transposed LDS reads: lane (r*4+cb) of each 16-lane group addresses
        // k-row kb+r, columns n+cb*4..; lane j then holds column n+j of rows kb..kb+3
        const int r = j16 >> 2, cb = j16 & 3;
        const int kb = ks * 16 + (q >> 1) * 8;
        const int n = wn * TN + ni * 32 + (q & 1) * 16 + cb * 4;
        const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
            (MLA_LDS bf16x4*)(&Bs[(kb + r) * OP_BLD + n]));
        const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
            (MLA_LDS bf16x4*)(&Bs[(kb + 4 + r) * OP_BLD + n]));
        bfr[ni] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      }
#pragma unroll
      for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
          acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[ni], af[mi], acc[mi][ni], 0, 0, 0);
    }
    __syncthreads();
    if (it + 1 < nk) {
      store_tiles();
      __syncthreads();
    }
  }

  // epilogue: the accumulators hold the transposed blocks, so a lane holds output
  // row l32 of each 32-row block and channels half*4 + 8i .. +3 of each
  // 32-channel block.  Each 32 x 32 block goes through this wave's part of the
  // (now idle) A buffer and comes back row-contiguous: 8 lanes cover one row's
  // 32 channels, so every z store instruction writes eight whole 128-byte lines
  // of f32 z (and each z_off read takes eight 64-byte runs).
  constexpr int SLD = 36;   // staged row: 32 floats + 4 of padding
  static_assert(NT / 64 * 32 * SLD * 4 <= OP_BM * OP_ALD * 2, "epilogue staging fits the A buffer");
  // lane quantities recomputed here rather than kept live across the K loop
  const int elane = (int)__lane_id();
  float MLA_LDS* stage = (float MLA_LDS*)As + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * (32 * SLD);
  // without z_off (every row protected) nothing is added: the lanes load from o_glob
  const bool has_zoff = a.z_off != nullptr;
  const uint16_t* zoff = (const uint16_t*)(has_zoff ? a.z_off : a.o_glob);
  const int prow = elane >> 3, pc4 = (elane & 7) * 4;   // read-back: row prow + 8p, channels pc4 .. +3
#pragma unroll
  for (int mi = 0; mi < MI; ++mi) {
    // the z_off this block adds (none on protected rows).  Every lane loads (element
    // 0 where nothing is added) and the unused values are zeroed after: no branch
    // around the loads, so each later wait counts exactly the loads still ahead of it.
    // Widened to f32 here, so that the block's one wait for its loads comes before any
    // of its stores (later waits would count those stores too).
    f32x4 addf[NI][4];
    {
      u32x2 addv[NI][4];
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          const int n = n0 + wn * TN + ni * 32 + pc4;
          const int r = wm * TM + mi * 32 + p * 8 + prow;
          const bool use = has_zoff && m0 + r < M && n < cw && !row_flag[r];
          const u32x2 zz = *(const u32x2*)(zoff + (use ? (int64_t)(m0 + r) * a.d_model + (int64_t)pg * cw + n : 0));
          addv[ni][p] = use ? zz : u32x2{0u, 0u};
        }
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          const u32x2 w = addv[ni][p];
          addf[ni][p] = f32x4{bf16_lo(w[0]), bf16_hi(w[0]), bf16_lo(w[1]), bf16_hi(w[1])};
        }
    }
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        *(f32x4 MLA_LDS*)(stage + (elane & 31) * SLD + (elane >> 5) * 4 + 8 * i) =
            f32x4{acc[mi][ni][4 * i], acc[mi][ni][4 * i + 1], acc[mi][ni][4 * i + 2], acc[mi][ni][4 * i + 3]};
      const int n = n0 + wn * TN + ni * 32 + pc4;   // 4 consecutive channels; cw is a multiple of 32
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const int rr = p * 8 + prow;
        f32x4 v = *(const f32x4 MLA_LDS*)(stage + rr * SLD + pc4);
        const int r = wm * TM + mi * 32 + rr;       // tile row
        if (m0 + r >= M || n >= cw) continue;
        const int64_t off = (int64_t)(m0 + r) * a.d_model + (int64_t)pg * cw + n;
        v += addf[ni][p];
        if (a.z_bf16)
          *(u32x2*)((uint16_t*)a.z + off) = u32x2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
        else
          *(f32x4*)(a.z + off) = v;
      }
    }
  }
}

// Pass L on the W_b kernel's plan (wb.hip): tiles of 32 MI protected rows x BN
// channels, 8 waves of 16 MI x BN / 4, operands by direct global->LDS loads 64 of K at a
// time into NST slices, the barrier between a step's halves.  The weight rows of a
// slice are K-major: channel fragments come by transposing reads.  The tile
// follows the device's count of protected rows (the host only knows the capacity),
// so one persistent workgroup per compute unit picks it and walks its tiles.
//
// At a few hundred protected rows the 256-row tiles of pass G left most of the chip
// idle in a serial K loop of 56 round trips.  Pass L at 310 protected rows 75 -> 25
// us, 2662 rows 129 -> 125, 16K rows with a rotary value 98 -> 73, 7291 rows 328 ->
// 296 (64 heads); 4014 rows of 128 heads 300 -> 254.
constexpr int OL_WAVES = 8, OL_GRID = 256;
constexpr int OL_LDS = 147456;                 // the largest variant's slices

// weight row of K index k of projection group pg's Local heads
__device__ __forceinline__ int local_w_row(const OprojArgs& a, int pg, int k) {
  const int hpg = a.n_heads / a.n_groups, gpp = a.n_groups / a.n_pg;
  const int kb = k / a.d_latent, d = k - kb * a.d_latent;
  const int gl = kb / (hpg - 1), j = kb - gl * (hpg - 1);
  const int gh = a.glob_head[pg * gpp + gl];
  return (gl * hpg + (j < gh ? j : j + 1)) * a.d_latent + d;
}

// MI: 16-row blocks per wave, BN: channels per tile (a wave's share: BN / 4), NST: slices
template <int MI, int BN, int NST>
__device__ __forceinline__ void local_tiles(const OprojArgs& a, int M, unsigned char* lds) {
  constexpr int NI = BN / 64, BM = 32 * MI;
  constexpr int LPR = BN / 8;                  // lanes, and 16-byte chunks, of a weight row
  constexpr int A_BYTES = BM * 128, STAGE = A_BYTES + 64 * BN * 2;
  constexpr int NA = A_BYTES / 1024, NLOADS = STAGE / 1024, LPW = (NLOADS + OL_WAVES - 1) / OL_WAVES;
  static_assert(NST * STAGE <= OL_LDS, "slices");
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hpg = a.n_heads / a.n_groups, gpp = a.n_groups / a.n_pg;
  const int cw = a.d_model / a.n_pg, DC = a.d_latent;
  const int K = gpp * (hpg - 1) * DC, nk = K / 64;
  const int64_t lda = (int64_t)a.n_groups * (hpg - 1) * DC;
  const int m_tiles = (M + BM - 1) / BM, n_tiles = (cw + BN - 1) / BN;
  // XCD x takes a contiguous range of tiles, row tiles innermost: neighbours share
  // a weight panel in its L2
  const int total = m_tiles * n_tiles * a.n_pg, per = (total + 7) / 8;
  const int wm = wave >> 2, wn = wave & 3, lg = lane >> 4, lc = lane & 15;

  for (int ti = (int)(blockIdx.x / 8); ti < per; ti += OL_GRID / 8) {
    int tb = (int)(blockIdx.x % 8) * per + ti;
    if (tb >= total) break;
    const int mt = tb % m_tiles;
    tb /= m_tiles;
    const int nt = tb % n_tiles, pg = tb / n_tiles;
    const int m0 = mt * BM, n0 = nt * BN;
    const unsigned char* A = (const unsigned char*)((const uint16_t*)a.o_loc + (int64_t)pg * K);
    const unsigned char* W = (const unsigned char*)((const uint16_t*)a.w_o + (int64_t)pg * (a.n_heads / a.n_pg) * DC * cw);

    // direct loads: load q fills LDS bytes [1024 q, +1024) of a stage.  q < NA: 8 rows
    // of the A slice, chunk c of row r at c ^ ((r >> 1) & 7), rows past the end repeat
    // the last.  The rest: weight rows k of BN channels, chunk c at c ^ 2 g(k),
    // g(k) = k % 4 + 4 (k / 8 % 2): the 8 rows a half-wave of a transposing read
    // touches hit distinct 32-byte bank groups; channels past the end repeat the last.
    const unsigned char* src[LPW];
    uint32_t voff[LPW];
#pragma unroll
    for (int j = 0; j < LPW; ++j) {
      const int q = std::min(wave + OL_WAVES * j, NLOADS - 1);
      if (q < NA) {
        const int r0 = 8 * q, lr = lane >> 3;
        const int first = std::min(r0, M - 1 - m0), row = std::min(r0 + lr, M - 1 - m0);
        src[j] = A + (int64_t)(m0 + first) * lda * 2;
        voff[j] = (uint32_t)((row - first) * lda * 2 + ((lane & 7) ^ (((r0 + lr) >> 1) & 7)) * 16);
      } else {
        const int k = 64 / LPR * (q - NA) + lane / LPR;
        const int c = (lane % LPR) ^ (2 * ((k & 3) | ((k >> 1) & 4)));
        src[j] = W;
        voff[j] = (uint32_t)(k * cw + std::min(n0 + c * 8, cw - 8)) * 2u;
      }
    }
    auto load_one = [&](int j, int kt, int64_t wk, int st) {
      const int q = std::min(wave + OL_WAVES * j, NLOADS - 1);
      dma16(src[j] + (q < NA ? (int64_t)kt * 128 : wk), voff[j], (const unsigned char MLA_LDS*)(lds + st + 1024 * q));
    };
    // byte offset of the next slice's first weight row: a slice never straddles two
    // heads, whose rows are consecutive
    int w_kt = 0, w_left = 0;
    int64_t w_at = 0;
    const int64_t w_step = (int64_t)64 * cw * 2;
    auto next_w = [&]() -> int64_t {
      if (w_left == 0) {
        w_at = (int64_t)local_w_row(a, pg, w_kt * 64) * cw * 2;
        w_left = DC / 64;
      } else {
        w_at += w_step;
      }
      --w_left;
      ++w_kt;
      return w_at;
    };

    f32x4 acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    struct Frags {
      bf16x8 a[MI], b[NI];
    };
    const unsigned char MLA_LDS* L = (const unsigned char MLA_LDS*)lds;
    const int fa = (wm * (BM / 2) + lc) * 128 + ((lg ^ ((lc >> 1) & 7)) * 16);
    const int rr = (lane >> 2) & 3, cb = lane & 3;
    const int fb = A_BYTES + (lg * 8 + rr) * (BN * 2) + (((wn * (2 * NI) + (cb >> 1)) ^ (2 * (rr | ((lg & 1) << 2)))) * 16) + (cb & 1) * 8;
    auto frag_a = [&](int st, int h, int i) -> bf16x8 { return *(const bf16x8 MLA_LDS*)(L + ((st + fa) ^ (h * 64)) + i * 2048); };
    auto frag_b = [&](int st, int h, int j) -> bf16x8 {
      const unsigned char MLA_LDS* p = L + ((st + fb) ^ (j * 32)) + h * (32 * BN * 2);
      const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((MLA_LDS bf16x4*)p);
      const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((MLA_LDS bf16x4*)(p + 4 * BN * 2));
      return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    };
    auto half = [&](const Frags& f, Frags& nx, int nst, int nh, auto LOAD, int kt, int64_t wk, int lst) {
      constexpr int R = MI + NI, PER = (R + MI - 1) / MI;
      int rd = 0, ld = 0;
#pragma unroll
      for (int i = 0; i < MI; ++i) {
#pragma unroll
        for (int k = 0; k < PER; ++k, ++rd)
          if (rd < NI) nx.b[rd] = frag_b(nst, nh, rd);
          else if (rd < R) nx.a[rd - NI] = frag_a(nst, nh, rd - NI);
        if constexpr (decltype(LOAD)::value) {
#pragma unroll
          for (int k = 0; k < (LPW + MI - 1) / MI; ++k, ++ld)
            if (ld < LPW) load_one(ld, kt, wk, lst);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int jj = 0; jj < NI; ++jj) {
          const int j = i & 1 ? NI - 1 - jj : jj;
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.b[j], f.a[i], acc[i][j], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    };
#pragma unroll
    for (int p = 0; p < NST; ++p)
      if (p < nk) {
        const int64_t wk = next_w();
#pragma unroll
        for (int j = 0; j < LPW; ++j) load_one(j, p, wk, p * STAGE);
      }
    if (nk >= NST) dma_barrier<(NST - 1) * LPW>(); else dma_barrier<0>();
    Frags f0, f1;
#pragma unroll
    for (int j = 0; j < NI; ++j) f0.b[j] = frag_b(0, 0, j);
#pragma unroll
    for (int i = 0; i < MI; ++i) f0.a[i] = frag_a(0, 0, i);
    int st = 0, kt = 0;
    for (; kt + NST < nk; ++kt) {
      const int64_t wk = next_w();
      half(f0, f1, st, 1, std::false_type{}, 0, 0, 0);
      dma_barrier<(NST - 2) * LPW>();
      const int nst = st == (NST - 1) * STAGE ? 0 : st + STAGE;
      half(f1, f0, nst, 0, std::true_type{}, kt + NST, wk, st);
      st = nst;
    }
    for (; kt < nk; ++kt) {
      half(f0, f1, st, 1, std::false_type{}, 0, 0, 0);
      dma_barrier<0>();
      const int nst = st == (NST - 1) * STAGE ? 0 : st + STAGE;
      half(f1, f0, nst, 0, std::false_type{}, 0, 0, 0);   // after the last slice: stale, not used
      st = nst;
    }

    // epilogue: 16 rows x BN / 4 channels a wave at a time through LDS (16-byte chunk c of
    // row r at c ^ (r & 7)), read back row-contiguous; the row's z is added in f32
    constexpr int CPR = 4 * NI, RPP = 64 / CPR, NP = 16 / RPP;   // chunks of a row, rows a pass, passes
    int orow[MI][NP];
    const int rl = lane / CPR, cl = lane % CPR;
    const int n = n0 + wn * (16 * NI) + cl * 4;   // cw is a multiple of 32
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        const int m = m0 + wm * (BM / 2) + i * 16 + p * RPP + rl;
        const int r = a.prot_rows[std::min(m, M - 1)];
        orow[i][p] = m < M && n < cw && r >= 0 && r < a.n_rows ? r : -1;   // outside z: skipped
      }
    dma_barrier<0>();
    unsigned char MLA_LDS* sw = (unsigned char MLA_LDS*)lds + wave * 8192;
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      f32x4 old[NP];
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        const int64_t off = orow[i][p] >= 0 ? (int64_t)orow[i][p] * a.d_model + (int64_t)pg * cw + n : 0;
        if (a.z_bf16) {
          const u32x2 w = *(const u32x2*)((const uint16_t*)a.z + off);
          old[p] = f32x4{bf16_lo(w[0]), bf16_hi(w[0]), bf16_lo(w[1]), bf16_hi(w[1])};
        } else {
          old[p] = *(const f32x4*)(a.z + off);
        }
      }
      unsigned char MLA_LDS* sb = sw + (i & 1) * 4096;
#pragma unroll
      for (int j = 0; j < NI; ++j) *(f32x4 MLA_LDS*)(sb + lc * (16 * CPR) + (((j * 4 + lg) ^ (lc & 7)) * 16)) = acc[i][j];
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        const int r = p * RPP + rl;
        f32x4 v = *(const f32x4 MLA_LDS*)(sb + r * (16 * CPR) + ((cl ^ (r & 7)) * 16));
        if (orow[i][p] < 0) continue;
        v += old[p];
        const int64_t off = (int64_t)orow[i][p] * a.d_model + (int64_t)pg * cw + n;
        if (a.z_bf16)
          *(u32x2*)((uint16_t*)a.z + off) = u32x2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
        else
          *(f32x4*)(a.z + off) = v;
      }
    }
    dma_barrier<0>();   // the next tile's slices may come in
  }
}

__global__ __launch_bounds__(OL_WAVES * 64, 2) void oproj_local_kernel(OprojArgs a) {
  __shared__ __attribute__((aligned(1024))) unsigned char lds[OL_LDS];
  // protected rows in use: the host count, or the device count clamped to the capacity
  int M = a.n_prot;
  if (a.n_prot_dev != nullptr) {
    const int d = *a.n_prot_dev;
    M = d < 0 ? 0 : (d < M ? d : M);
  }
  if (M == 0) return;
  const int cw = a.d_model / a.n_pg;
  const int64_t n256 = (int64_t)((cw + 255) / 256) * a.n_pg, n128 = (int64_t)((cw + 127) / 128) * a.n_pg;
  // The tile whose rounds over the chip cost least.  Heights 32 mi of 256 channels as
  // in wb.hip, a tile taken as mi + 3 (here in thirds).  While a round is not full a
  // compute unit's direct loads are what a slice waits for, so tiles of 128 channels,
  // 20 or 24 KB a slice against 36 for 32 x 256: at K = 3584, 4096 channels 19.7 and
  // 21.8 us against 30.8 at 32 rows, and 64 x 128 25 against 33 at 310 (two rounds of
  // 32 x 128: 38), 27 against 36 at 512; at 600 rows 64 x 128 takes two rounds, 45,
  // and 64 x 256 one, 38.
  int best = 8;
  int64_t cost = INT64_MAX;
  auto tile = [&](int id, int bm, int64_t nt, int w) {
    const int64_t c = (((int64_t)M + bm - 1) / bm * nt + OL_GRID - 1) / OL_GRID * w;
    if (c < cost) {
      cost = c;
      best = id;
    }
  };
  tile(8, 256, n256, 33);
  tile(4, 128, n256, 21);
  tile(2, 64, n256, 15);
  tile(12, 64, n128, 9);
  tile(11, 32, n128, 8);
  best = __builtin_amdgcn_readfirstlane(best);
  if (best == 11)
    local_tiles<1, 128, 7>(a, M, lds);
  else if (best == 12)
    local_tiles<2, 128, 6>(a, M, lds);
  else if (best == 2)
    local_tiles<2, 256, 3>(a, M, lds);
  else if (best == 4)
    local_tiles<4, 256, 3>(a, M, lds);
  else
    local_tiles<8, 256, 2>(a, M, lds);
}

// W_{a,L}^T of each projection group, for the producer's Local projection as a
// plain K-contiguous GEMM: wt[pg][n][k] = w_o[pg][row(k)][n], k running over the
// Local heads of pg's groups in the order of the head outputs' columns (ascending
// head index, the group's Global head skipped).  64 x 64 tiles through LDS, so
// that both the reads (along n) and the writes (along k) are row-contiguous.
__global__ __launch_bounds__(256) void local_wt_kernel(OprojArgs a, uint16_t* wt, int n_ktiles, int n_ntiles) {
  __shared__ uint16_t tile[64][65];
  const int hpg = a.n_heads / a.n_groups, gpp = a.n_groups / a.n_pg;
  const int cw = a.d_model / a.n_pg, DC = a.d_latent;
  const int heads_pp = a.n_heads / a.n_pg;
  const int64_t KL = (int64_t)gpp * (hpg - 1) * DC;
  int b = blockIdx.x;
  const int kt = b % n_ktiles;
  b /= n_ktiles;
  const int nt = b % n_ntiles;
  const int pg = b / n_ntiles;
  const uint16_t* W = (const uint16_t*)a.w_o + (int64_t)pg * heads_pp * DC * cw;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  for (int r = ty; r < 64; r += 4) {   // read: tile row r = k, column tx = n
    const int64_t k = (int64_t)kt * 64 + r;
    const int n = nt * 64 + tx;
    uint16_t v = 0;
    if (k < KL && n < cw) {
      v = W[(int64_t)local_w_row(a, pg, (int)k) * cw + n];
    }
    tile[r][tx] = v;
  }
  __syncthreads();
  for (int r = ty; r < 64; r += 4) {   // write: row n, column k
    const int n = nt * 64 + r;
    const int64_t k = (int64_t)kt * 64 + tx;
    if (n < cw && k < KL) wt[((int64_t)pg * cw + n) * KL + k] = tile[tx][r];
  }
}

hipError_t launch_local_wt(const OprojArgs& a, uint16_t* wt, hipStream_t s) {
  const int hpg = a.n_heads / a.n_groups, gpp = a.n_groups / a.n_pg;
  const int64_t KL = (int64_t)gpp * (hpg - 1) * a.d_latent;
  const int cw = a.d_model / a.n_pg;
  const int n_ktiles = (int)((KL + 63) / 64), n_ntiles = (cw + 63) / 64;
  const int64_t blocks = (int64_t)n_ktiles * n_ntiles * a.n_pg;
  if (blocks == 0) return hipSuccess;
  local_wt_kernel<<<dim3((unsigned)blocks), dim3(256), 0, s>>>(a, wt, n_ktiles, n_ntiles);
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void fill_zero_kernel(u32x4* p, int64_t n16) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = u32x4{0u, 0u, 0u, 0u};
}

// zero fill with a kernel (no memset node, so the call can be graph-captured);
// p is 16-byte aligned and bytes a multiple of 16
hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t s) {
  const int64_t n16 = (int64_t)(bytes / 16);
  if (n16 == 0) return hipSuccess;
  const unsigned blocks = (unsigned)std::min<int64_t>((n16 + 255) / 256, 16384);
  fill_zero_kernel<<<dim3(blocks), dim3(256), 0, s>>>((u32x4*)p, n16);
  return hipGetLastError();
}

// 256 x 128 tiles, 8 waves (4 x 2 wave tiles of 64 x 64): 58 KB of LDS and up to
// 128 registers per wave, two workgroups per CU.  Same per-element K order as any
// other tile shape, so the results do not depend on it.  At 256K the step's two
// passes, when both ran on such tiles, took 3.16 ms (128 x 256 the same; 256 x 256 with one workgroup per CU
// 3.58, 64 x 256 with three 3.39, 128 x 128 with four 4.03 ms).
constexpr int kOpBM = 256, kOpBN = 128, kOpWM = 4, kOpWN = 2;

int64_t oproj_workgroups(int64_t M, int d_model, int n_pg) {
  const int64_t tiles = (M + kOpBM - 1) / kOpBM * ((d_model / n_pg + kOpBN - 1) / kOpBN) * n_pg;
  return 8 * ((tiles + 7) / 8);
}

hipError_t launch_oproj(const OprojArgs& a, hipStream_t s) {
  if (a.n_rows > 0) {
    const int cw = a.d_model / a.n_pg;
    const int n_tiles = (cw + kOpBN - 1) / kOpBN, m_tiles = (int)((a.n_rows + kOpBM - 1) / kOpBM);
    const int total = m_tiles * n_tiles * a.n_pg;
    oproj_kernel<kOpBM, kOpBN, kOpWM, kOpWN><<<dim3((unsigned)(8 * ((total + 7) / 8))), dim3(kOpWM * kOpWN * 64), 0, s>>>(
        a, m_tiles, n_tiles);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (a.n_prot > 0 && a.n_heads > a.n_groups) {
    oproj_local_kernel<<<dim3(OL_GRID), dim3(OL_WAVES * 64), 0, s>>>(a);
    return hipGetLastError();
  }
  return hipSuccess;
}

}  // namespace mla
