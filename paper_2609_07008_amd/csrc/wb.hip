// Shared second output projection y = W_b z (Sec. 2.1 eq:factorization; Alg. 2
// returns W_b z): every row's group-sliced state z [N, d_in] meets the one
// dense W_b, stored as a linear layer's weight [d_out, d_in].  Both operands are
// K-contiguous, so this is C = A B^T with A = z, B = W_b, on bf16 MFMA with fp32
// accumulation; y is written in fp32 or bf16.
//
// Tiles of 32 MI rows x BN channels (256; 128 while a round over the chip is not full,
// and for narrow outputs) per workgroup of 8 waves (2 x 4, each 16 MI x BN / 4); the
// operands come in by direct global->LDS loads, 64 of K at a time, NST slices in LDS.  On a full chip power is what bounds it: 16x16x32 MFMAs take less
// per flop than 32x32x16 (see attend_pair.hip), so a wave's 16-row fragments feed
// MI x 4 of them, neighbours sharing an operand.  What stalls it otherwise is the
// barrier of a slice: it sits between a step's two halves, so that a half's MFMAs,
// their fragments already in registers, run over the LDS reads of the next half and
// over the direct loads, which all eight waves issue a few at a time.  The output
// leaves through LDS as whole 128-byte lines (32-byte runs cost 9 % of the call).
// Tile order: workgroups go to the 8 XCDs round-robin, so XCD x takes a contiguous
// range of tiles, and inside it tiles walk 8 row panels per column panel, so tiles
// resident together on an XCD share A and B panels in its L2 (4 panels 1 % slower,
// 2 or 16 7-14 %).
//
// 264,192 rows, 4096 -> 4096: bf16 y 7.10 -> 6.37 ms (1.39 PFLOP/s), f32 y 7.40 ->
// 6.86; 2100 rows f32 81 -> 66 us, 300 rows 76 -> 21, 16 rows 72 -> 8.
//
// Every tile and the few-row kernel add an element's products in the same order: a row of
// y does not depend on how many rows the call has.
#include "wb.h"

#include <algorithm>
#include <type_traits>

namespace mla {
namespace {

constexpr int WB_BK = 64;
constexpr int WB_WAVES = 8;                           // 2 x 4 waves of (BM/2) x (BN/4)
constexpr int WB_ROWB = WB_BK * 2;                    // bytes of one row of a slice
constexpr int64_t kWbFewRows = 32, kWbFewBlocks = 512;   // largest requests of the few-row kernel
constexpr int WB_GM = 8;                              // row panels per column panel in the tile walk

__device__ __forceinline__ int swz(int r) { return (r >> 1) & 7; }

// MI: 16-row blocks per wave (tile of 32 MI rows x BN channels); NST: K slices in LDS
template <bool OUT_BF16, int MI, int BN, int NST>
__global__ __launch_bounds__(WB_WAVES * 64, 2) void wb_gemm_kernel(WbArgs a, int m_tiles, int n_tiles, bool stream_out) {
  constexpr int NI = BN / 64, BM = 32 * MI;
  constexpr int A_BYTES = BM * WB_ROWB, STAGE = A_BYTES + BN * WB_ROWB;
  constexpr int NLOADS = STAGE / 1024;                       // 1 KB direct loads (8 rows each) per slice
  constexpr int LPW = (NLOADS + WB_WAVES - 1) / WB_WAVES;    // per wave; past the end the last one again
  __shared__ __attribute__((aligned(1024))) unsigned char lds[NST * STAGE];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  // XCD-aware, grouped tile walk (batches one after another)
  const int per_batch = m_tiles * n_tiles;
  const int total = per_batch * a.batch;
  const int per = (total + 7) / 8;
  const int tb = (int)(blockIdx.x % 8) * per + (int)(blockIdx.x / 8);
  if ((int)(blockIdx.x / 8) >= per || tb >= total) return;
  const int bt = tb / per_batch, t = tb % per_batch;
  const int group = t / (WB_GM * n_tiles), rem = t % (WB_GM * n_tiles);
  const int gm = std::min(WB_GM, m_tiles - group * WB_GM);
  const int mt = group * WB_GM + rem % gm, nt = rem / gm;
  const int64_t m0 = (int64_t)mt * BM;
  const int n0 = nt * BN;

  // Direct loads: load q of a slice fills LDS bytes [1024 q, +1024) of the stage, the
  // slice's A rows then its B rows, 8 rows each; row r's chunk c sits at slot c ^
  // swz(r).  A load takes a wave-uniform base (its first row) plus a 32-bit lane
  // offset within its 8 rows.  Rows past the end are clamped to the last one (their
  // results are not stored).
  const int64_t ldz = a.ldz, ldw = a.ldw;
  const unsigned char* src[LPW];
  uint32_t voff[LPW];
  int dst[LPW];
#pragma unroll
  for (int j = 0; j < LPW; ++j) {
    const int q = std::min(wave + WB_WAVES * j, NLOADS - 1);
    const bool is_a = q < A_BYTES / 1024;
    const int r0 = 8 * (is_a ? q : q - A_BYTES / 1024), lr = lane >> 3;
    const int64_t rows = is_a ? a.n_rows - m0 : (int64_t)a.d_out - n0;   // rows from the tile's first to the last
    const int64_t first = std::min<int64_t>(r0, rows - 1), row = std::min<int64_t>(r0 + lr, rows - 1);
    const int64_t ld = is_a ? ldz : ldw;
    src[j] = (const unsigned char*)(is_a ? a.z + bt * a.z_batch : a.w_b + bt * a.w_batch) + ((is_a ? m0 : n0) + first) * ld * 2;
    voff[j] = (uint32_t)((row - first) * ld * 2 + ((lane & 7) ^ swz(r0 + lr)) * 16);
    dst[j] = 1024 * q;
  }
  auto load_one = [&](int j, int kt, int st) {
    dma16(src[j] + (int64_t)kt * WB_ROWB, voff[j], (const unsigned char MLA_LDS*)(lds + st + dst[j]));
  };

  f32x4 acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // fragments (16 rows x 32 of K): lane group lg holds chunk 4 h + lg of row lc; the
  // rows' swizzle repeats every 16, so blocks are immediate offsets
  const int wm = wave >> 2, wn = wave & 3, lg = lane >> 4, lc = lane & 15;
  const int fa = (wm * (BM / 2) + lc) * WB_ROWB + ((lg ^ swz(lc)) * 16);
  const int fb = A_BYTES + (wn * (BN / 4) + lc) * WB_ROWB + ((lg ^ swz(lc)) * 16);
  struct Frags {
    bf16x8 a[MI], b[NI];
  };
  auto frag = [&](int base, int st, int h, int i) -> bf16x8 {
    return *(const bf16x8 MLA_LDS*)((const unsigned char MLA_LDS*)lds + ((st + base) ^ (h * 64)) + i * 16 * WB_ROWB);
  };
  // the MFMAs of one 32-wide half step, and beside them the next half's fragment
  // reads and (LOAD) the direct loads of a later slice.  The transposed tile: a lane
  // holds output row lc and four consecutive channels of each block.
  auto half = [&](const Frags& f, Frags& nx, int nst, int nh, auto LOAD, int kt, int lst) {
    constexpr int R = MI + NI;                 // fragments to read, spread over the rows of MFMAs
    constexpr int PER = (R + MI - 1) / MI;
    int rd = 0, ld = 0;
#pragma unroll
    for (int i = 0; i < MI; ++i) {
#pragma unroll
      for (int k = 0; k < PER; ++k, ++rd)
        if (rd < NI) nx.b[rd] = frag(fb, nst, nh, rd);
        else if (rd < R) nx.a[rd - NI] = frag(fa, nst, nh, rd - NI);
      if constexpr (decltype(LOAD)::value) {
#pragma unroll
        for (int k = 0; k < (LPW + MI - 1) / MI; ++k, ++ld)
          if (ld < LPW) load_one(ld, kt, lst);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int jj = 0; jj < NI; ++jj) {
        const int j = i & 1 ? NI - 1 - jj : jj;   // neighbours share an operand
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.b[j], f.a[i], acc[i][j], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // Slices 0 .. NST-1 go out first.  Step kt: the first half's MFMAs beside the reads
  // of the second half's fragments; one barrier (slice kt is read by every wave, so
  // its buffer is free; slice kt + 1 has landed); the second half's MFMAs beside the
  // loads of slice kt + NST and the reads of slice kt + 1's first half.
  const int nk = a.d_in / WB_BK;
#pragma unroll
  for (int p = 0; p < NST; ++p)
    if (p < nk)
#pragma unroll
      for (int j = 0; j < LPW; ++j) load_one(j, p, p * STAGE);
  if (nk >= NST) dma_barrier<(NST - 1) * LPW>(); else dma_barrier<0>();
  Frags f0, f1;
#pragma unroll
  for (int j = 0; j < NI; ++j) f0.b[j] = frag(fb, 0, 0, j);
#pragma unroll
  for (int i = 0; i < MI; ++i) f0.a[i] = frag(fa, 0, 0, i);
  int st = 0, kt = 0;
  for (; kt + NST < nk; ++kt) {
    half(f0, f1, st, 1, std::false_type{}, 0, 0);
    dma_barrier<(NST - 2) * LPW>();
    const int nst = st == (NST - 1) * STAGE ? 0 : st + STAGE;
    half(f1, f0, nst, 0, std::true_type{}, kt + NST, st);
    st = nst;
  }
  for (; kt < nk; ++kt) {
    half(f0, f1, st, 1, std::false_type{}, 0, 0);
    dma_barrier<0>();
    const int nst = st == (NST - 1) * STAGE ? 0 : st + STAGE;
    half(f1, f0, nst, 0, std::false_type{}, 0, 0);   // after the last slice: reads of a stale buffer, not used
    st = nst;
  }

  // Epilogue through LDS, 16 rows x BN / 4 channels a wave at a time: written in the
  // accumulator layout (row lc, channels lg*4 .. +3 of each block; 16-byte chunk c
  // of row r at c ^ (r & SW)), read back row-contiguous, so that each store writes
  // whole 128-byte lines.
  dma_barrier<0>();
  constexpr int ES = OUT_BF16 ? 2 : 4, ROW = BN / 4 * ES;   // element and row bytes
  constexpr int CH = ROW / 16, RPI = 64 / CH;           // 16-byte chunks a row, rows a store
  constexpr int SW = CH < 8 ? CH - 1 : 7;
  unsigned char MLA_LDS* sw = (unsigned char MLA_LDS*)lds + wave * (2 * 16 * ROW);
  const int64_t ybase = bt * a.y_batch;
  // whole chunks: y is 16-byte aligned
  const bool vec = ((a.ldy | a.y_batch) & (16 / ES - 1)) == 0;
  const int rl = lane / CH, cl = lane % CH;
  const int n = n0 + wn * (BN / 4) + cl * (16 / ES);
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    unsigned char MLA_LDS* sb = sw + (i & 1) * (16 * ROW);
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const f32x4 v = acc[i][j];
      if (OUT_BF16)
        *(u32x2 MLA_LDS*)(sb + lc * ROW + (((j * 2 + (lg >> 1)) ^ (lc & SW)) * 16) + (lg & 1) * 8) =
            u32x2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
      else
        *(f32x4 MLA_LDS*)(sb + lc * ROW + (((j * 4 + lg) ^ (lc & SW)) * 16)) = v;
    }
#pragma unroll
    for (int p = 0; p < 16 / RPI; ++p) {
      const int r = p * RPI + rl;
      const u32x4 v = *(const u32x4 MLA_LDS*)(sb + r * ROW + ((cl ^ (r & SW)) * 16));
      const int64_t m = m0 + wm * (BM / 2) + i * 16 + r;
      if (m >= a.n_rows) continue;
      const int64_t at = ybase + m * a.ldy + n;
      if (vec && n + 16 / ES <= a.d_out) {
        u32x4* q = (u32x4*)((unsigned char*)a.y + at * ES);
        if (stream_out) __builtin_nontemporal_store(v, q); else *q = v;
      } else {
#pragma unroll
        for (int e = 0; e < 16 / ES; ++e) {
          if (n + e >= a.d_out) continue;
          if (OUT_BF16)
            ((uint16_t*)a.y)[at + e] = (uint16_t)(v[e / 2] >> (16 * (e & 1)));
          else
            ((uint32_t*)a.y)[at + e] = v[e];
        }
      }
    }
  }
}

// Few rows (a query block, a chunk of new tokens): the weight is read once, so what
// counts is how much of it is in flight.  A workgroup takes 16 output channels and up
// to 16 MB rows (all of them); its 8 waves bring 512 of K at a time, a kilobyte of one
// weight or z row a direct load, into NST stages (128 KB at 16 rows, 144 KB at 32) and
// wave b < MB runs the MFMAs of row block b, one after the other over K: the sum of an
// element has the order it has in the tiles, so a row of y has the same bits whatever
// the number of rows.  Chunk c of row r sits at c ^ (r & 15).
// 4096 -> 4096: 7.7 us at 1 row, 7.4 at 16, 9.1 at 32 (K split over the waves, fragments
// straight from memory: 8.2, 11.4, 16.3); 16384 -> 4096 28, 29, 33 us (27, 35, 48).
template <bool OUT_BF16, int MB, int NST>
__global__ __launch_bounds__(WB_WAVES * 64) void wb_rows_kernel(WbArgs a, int n_blocks) {
  constexpr int BK = 512, ROWB = BK * 2, ROWS = 16 + 16 * MB, STAGE = ROWS * ROWB;
  constexpr int LPW = ROWS / WB_WAVES;           // 1 KB direct loads per wave and stage
  static_assert(ROWB == 1024 && ROWS % WB_WAVES == 0, "a load takes a row");
  __shared__ __attribute__((aligned(1024))) unsigned char lds[NST * STAGE];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lg = lane >> 4, lc = lane & 15;
  const int bt = blockIdx.x / n_blocks, n0 = (int)(blockIdx.x % n_blocks) * 16;
  // rows past the end repeat the last one; their results are not stored
  const unsigned char* src[LPW];
#pragma unroll
  for (int j = 0; j < LPW; ++j) {
    const int r = wave * LPW + j;
    src[j] = (const unsigned char*)(r < 16 ? a.w_b + bt * a.w_batch + (int64_t)std::min(n0 + r, a.d_out - 1) * a.ldw
                                           : a.z + bt * a.z_batch + std::min<int64_t>(r - 16, a.n_rows - 1) * a.ldz);
  }
  auto load = [&](int s, int st) {   // past the end of K: the last chunk again, not used
#pragma unroll
    for (int j = 0; j < LPW; ++j) {
      const int r = wave * LPW + j;
      const uint32_t at = std::min((uint32_t)(s * ROWB + (lane ^ (r & 15)) * 16), (uint32_t)(a.d_in * 2 - 16));
      dma16(src[j], at, (const unsigned char MLA_LDS*)(lds + st + r * ROWB));
    }
  };
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  const unsigned char MLA_LDS* L = (const unsigned char MLA_LDS*)lds;
  const int nk = a.d_in / 32, ns = (a.d_in + BK - 1) / BK;
#pragma unroll
  for (int p = 0; p < NST - 1; ++p) load(p, p * STAGE);
  int st = 0;
  for (int s = 0; s < ns; ++s) {
    // stage s has landed, and every wave has read stage s - 1, whose buffer is next
    dma_barrier<(NST - 2) * LPW>();
    load(s + NST - 1, st == 0 ? (NST - 1) * STAGE : st - STAGE);
    if (wave < MB) {
      const unsigned char MLA_LDS* pw = L + st + lc * ROWB;
      const unsigned char MLA_LDS* pz = L + st + (16 + wave * 16 + lc) * ROWB;
      const int left = nk - s * (BK / 32);
      constexpr int N = BK / 32, AHEAD = 4;   // fragments read ahead of their MFMA
      bf16x8 fw[N], fz[N];
      auto frag = [&](int k) {
        const int o = ((k * 4 + lg) ^ lc) * 16;
        fw[k] = *(const bf16x8 MLA_LDS*)(pw + o);
        fz[k] = *(const bf16x8 MLA_LDS*)(pz + o);
      };
#pragma unroll
      for (int k = 0; k < AHEAD; ++k) frag(k);
#pragma unroll
      for (int k = 0; k < N; ++k) {
        if (k + AHEAD < N) frag(k + AHEAD);
        __builtin_amdgcn_sched_barrier(0);
        if (k < left) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[k], fz[k], acc, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    st = st == (NST - 1) * STAGE ? 0 : st + STAGE;
  }
  dma_barrier<0>();   // the loads past the end have landed
  if (wave >= MB) return;
  const int64_t m = wave * 16 + lc;
  if (m >= a.n_rows) return;
  const int64_t at = bt * a.y_batch + m * a.ldy + n0 + lg * 4;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    if (n0 + lg * 4 + e >= a.d_out) continue;
    if (OUT_BF16)
      ((__bf16*)a.y)[at + e] = (__bf16)acc[e];
    else
      ((float*)a.y)[at + e] = acc[e];
  }
}

template <bool OUT_BF16>
hipError_t launch_rows(const WbArgs& a, hipStream_t s) {
  const int n_blocks = (a.d_out + 15) / 16;
  const unsigned gx = (unsigned)(n_blocks * a.batch);
  if (a.n_rows <= 16)
    wb_rows_kernel<OUT_BF16, 1, 4><<<dim3(gx), dim3(WB_WAVES * 64), 0, s>>>(a, n_blocks);
  else
    wb_rows_kernel<OUT_BF16, 2, 3><<<dim3(gx), dim3(WB_WAVES * 64), 0, s>>>(a, n_blocks);
  return hipGetLastError();
}

template <bool OUT_BF16, int MI, int BN, int NST>
hipError_t launch_tiles(const WbArgs& a, hipStream_t s) {
  const int m_tiles = (int)((a.n_rows + 32 * MI - 1) / (32 * MI));
  const int n_tiles = (a.d_out + BN - 1) / BN;
  const int total = m_tiles * n_tiles * a.batch;
  // an output beyond the L2s' 32 MB cannot stay there: stored past them, it leaves
  // them to the panels (33,792 rows f32: 927 -> 882 us; 264,192 rows bf16: 6.39 -> 6.31 ms)
  const bool stream_out = a.n_rows * a.d_out * a.batch * (OUT_BF16 ? 2 : 4) > (int64_t)32 << 20;
  wb_gemm_kernel<OUT_BF16, MI, BN, NST><<<dim3((unsigned)(8 * ((total + 7) / 8))), dim3(WB_WAVES * 64), 0, s>>>(a, m_tiles, n_tiles, stream_out);
  return hipGetLastError();
}

template <bool OUT_BF16>
hipError_t launch_out(const WbArgs& a, hipStream_t s) {
  // Up to 32 rows and 512 workgroups of 16 channels, two rounds over the compute units,
  // the few-row kernel: 4096 -> 4096 7.8 us at 1 row, 8.9 at 32 (tiles 16.4, 17.3), -> 8192
  // 15.3, 18.5 (17.2, 17.6), 1024 -> 8192 7.6, 7.7 (7.9, 8.3).  Wider outputs fill the chip
  // with tiles, which read z once for 128 channels: 4096 -> 12288 17.9, 19.0 us against
  // 22.0, 27.0, -> 32768 42.8, 43.8 against 51.5, 63.7.
  const int64_t few_blocks = ((int64_t)a.d_out + 15) / 16 * a.batch;
  if (a.n_rows <= kWbFewRows && few_blocks <= kWbFewBlocks) return launch_rows<OUT_BF16>(a, s);
  // The tile whose rounds over the 256 compute units cost least.  256 channels: 32 mi
  // rows taken as mi + 3 (here in thirds; one round at K = 4096, heights 1 .. 8: 28,
  // 34, 42, 48, 56, 63, 73, 74 us).  While a round is not full a slice waits for its
  // unit's direct loads, 36 KB for 32 x 256, so there are tiles of 128 channels, 20 to
  // 32 KB (17.7, 19.6, 24.6, 25.5 us).  At 4096 channels: 128 rows 18.2 us at 32 x 128
  // against 28 at 32 x 256, 500 rows 23 at 64 x 128 against 31, 1024 rows 35.5 at 128 x
  // 128 against 38.6 at 64 x 256; 2100 rows 68 at 160 x 256 against 82 at height 256,
  // 33,792 rows 849 at 256 x 256 against 875 at 192.
  int best = 8;
  int64_t cost = INT64_MAX;
  auto tile = [&](int id, int mi, int bn, int w) {
    const int64_t tiles = (a.n_rows + 32 * mi - 1) / (32 * mi) * ((a.d_out + bn - 1) / bn) * a.batch;
    const int64_t c = (tiles + 255) / 256 * w;
    if (c < cost) {
      cost = c;
      best = id;
    }
  };
  for (int mi = 8; mi >= 2; --mi) tile(mi, mi, 256, 3 * (mi + 3));
  for (int mi = 4; mi >= 1; --mi) tile(10 + mi, mi, 128, mi + 7);
  switch (best) {
    case 2: return launch_tiles<OUT_BF16, 2, 256, 3>(a, s);
    case 3: return launch_tiles<OUT_BF16, 3, 256, 3>(a, s);
    case 4: return launch_tiles<OUT_BF16, 4, 256, 3>(a, s);
    case 5: return launch_tiles<OUT_BF16, 5, 256, 3>(a, s);
    case 6: return launch_tiles<OUT_BF16, 6, 256, 2>(a, s);
    case 7: return launch_tiles<OUT_BF16, 7, 256, 2>(a, s);
    case 11: return launch_tiles<OUT_BF16, 1, 128, 7>(a, s);
    case 12: return launch_tiles<OUT_BF16, 2, 128, 6>(a, s);
    case 13: return launch_tiles<OUT_BF16, 3, 128, 5>(a, s);
    case 14: return launch_tiles<OUT_BF16, 4, 128, 4>(a, s);
    default: return launch_tiles<OUT_BF16, 8, 256, 2>(a, s);
  }
}

}  // namespace

hipError_t launch_wb(const WbArgs& a, hipStream_t s) {
  if (a.n_rows == 0) return hipSuccess;
  return a.y_bf16 ? launch_out<true>(a, s) : launch_out<false>(a, s);
}

}  // namespace mla
