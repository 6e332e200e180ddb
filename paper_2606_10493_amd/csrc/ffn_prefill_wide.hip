// Prefill-regime expert FFN, wide tiles: the block-scaled FP8 grouped GEMM of
// ffn_prefill.hip over 256 weight rows x up to 256 expert rows per workgroup,
// for launches whose experts have enough rows (see prefill_tile_rows).  Every
// row's arithmetic is that kernel's (two chained MFMAs per 128-K block from
// zero, blocks promoted in order), so the results are the same bits.
//
// A 256 x 128 tile moves 48 KB into its CU per K block for 1024 matrix-core
// cycles, and the address path takes 57 bytes a clock: 840 cycles.  A 256 x 256
// tile moves 64 KB for 2048.  Its 128 accumulator registers leave no room for a
// register ring, so both operands go from global memory straight into LDS
// (two stages each), and the waves are 4 x 2 over 64 weight rows x 128 expert
// rows, which reads 94 bytes of LDS per matrix-core cycle instead of 125.
// Eight waves that a barrier keeps in step spend loads, LDS reads and MFMAs one
// after the other unless each is issued under another step's MFMAs; see the K
// loop.  One workgroup per CU takes tiles from queues (below): unequal tiles
// under skewed routing cost one XCD's fixed share several times another's.
//
// Measured (rocprofv3, H 7168, I 2048, 256 experts x 8, against 256 x 128
// tiles; gate/up, down): 4096 tokens 1669 -> 1491, 987 -> 932 us; 5000 tokens
// 1932 -> 1589, 1201 -> 1017; 6144 tokens 2007 -> 1757, 1340 -> 1130; 8192
// tokens 2466 -> 2329 (1.65 PFLOP/s), 1692 -> 1500 us; 8192 tokens, Zipf(1)
// routing 2502 -> 2411, 1743 -> 1524 us.  What remains: gate/up -14 %, down
// -14 % with every load in cache; -11 % without the promotion; the chip holds
// 1.9 - 2.0 GHz under it (the fp8 library GEMM: 1.88).
#include "ffn_prefill.h"

#include <math.h>

#include <algorithm>
#include <type_traits>

namespace moe {

namespace {

constexpr int kThreads = 512;                     // 8 waves: 4 of 64 weight rows x 2 halves of the expert rows
constexpr int kStageW = 256 * kBlock;             // one K block of the weights in LDS
constexpr int kStageA = kPrefillWideRows * kBlock;
constexpr int kScaleWin = 4;                      // K blocks per row-scale window
constexpr int kWideMaxBlocks = 64;                // K / 128 at most
constexpr int kWideWorkgroups = 256;              // one per CU (LDS and registers allow no more)
constexpr double kWideMinRounds = 2.4;            // full tiles per CU (see prefill_tile_rows)

struct Smem {
  uint8_t w[2][kStageW];                          // packed operand tiles, slot (16-row group) s at 2048 s
  uint8_t a[2][kStageA];                          // expert rows, 128-byte rows, chunks swizzled (swz)
  float sa[2][kPrefillWideRows][kScaleWin];       // row scales of four K blocks
  float sw[2][kWideMaxBlocks];                    // weight scales of the tile's two 128-row blocks
  int idx[kPrefillWideRows];                      // row index of tile row t (see row_index)
  int pos[kPrefillWideRows];                      // with row tables: sorted position of tile row t
  float rowmax[4][kPrefillWideRows];              // GATEUP: |h| maxima per weight-row quarter
  int next;                                       // the workgroup's next work item
};

// 64 lanes' dwords (lane l from src, its own address) to LDS lds + 4 l.
__device__ __forceinline__ void async_load_dwords(const void* src, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off"
               :
               : "s"(__builtin_amdgcn_readfirstlane((int)lds)), "v"(src)
               : "memory");
}

// One tile.
template <bool GATEUP>
__device__ __forceinline__ void wide_tile(const PrefillArgs p, Smem& sm, int item, int tid) {
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r32 = lane & 31, g2 = lane >> 5;
  const int wr = wave & 3, wc = wave >> 2;

  const Tile tile = tile_of(p, item);
  const int m0 = tile.m0, mc = tile.mc, nt = tile.nt;
  const int nb = p.K / kBlock;
  const int groups = (mc + 31) >> 5;                          // 1 .. 8
  const int grp0 = wc ? (groups + 1) >> 1 : 0;                // this wave's first group
  const int nq = wc ? groups >> 1 : (groups + 1) >> 1;        // and their number

  // Row indices (and positions, weight scales) go out first, then two K blocks
  // of weights, all straight into LDS.
  const int64_t ebase = (int64_t)tile.e * p.N * p.K;
  // This wave loads slots 2 wave and 2 wave + 1 of the weight tile.
  const uint8_t *w_lo, *w_hi;
  if (GATEUP) {
    const int64_t grp = (int64_t)nt * (kBlock / 16) + wave;
    w_lo = p.w0 + ebase + grp * nb * kTileBytes;
    w_hi = p.w1 + ebase + grp * nb * kTileBytes;
  } else {
    w_lo = p.w0 + ebase + ((int64_t)nt * (kPrefillWeightRows / 16) + 2 * wave) * nb * kTileBytes;
    w_hi = w_lo + (int64_t)nb * kTileBytes;
  }
  const uint32_t lds_w = lds_address(sm.w) + wave * 4096;
  auto load_weight = [&](int on, int blk, int i) {  // i = 0 .. 3
    async_load_1k_if(on, (i < 2 ? w_lo : w_hi) + (int64_t)blk * kTileBytes + (i & 1) * 1024, lane * 16,
                     lds_w + (blk & 1) * kStageW + i * 1024);
  };
  {
    const int32_t* rsrc = GATEUP ? (p.row_tok ? p.row_tok : p.sorted_src) : p.row_pos;
    const int t = (wave & 3) * 64 + lane;  // waves 0-3: tile rows; the tile's last row stands in past mc
    if (wave < 4) {
      if (rsrc) async_load_dwords(rsrc + m0 + min(t, mc - 1), lds_address(sm.idx) + wave * 256);
    } else {
      if (GATEUP && p.row_pos) async_load_dwords(p.row_pos + m0 + min(t, mc - 1), lds_address(sm.pos) + (wave - 4) * 256);
      if (wave < 6) {
        const int h = wave - 4;
        const int64_t wrow = (int64_t)tile.e * (p.N / kBlock) + (GATEUP ? nt : 2 * nt + h);
        async_load_dwords(((GATEUP && h) ? p.s1 : p.s0) + wrow * nb + min(lane, nb - 1), lds_address(sm.sw[h]));
      }
    }
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) load_weight(1, i >> 2, i & 3);  // nb >= 4
  wait_async_and_barrier<8>();  // the indices; the weights stay in flight

  // The A row of tile row t: its token (GATEUP) or sorted position; -1 if the
  // index is out of range.
  auto row_index = [&](int t) {
    int v;
    if (GATEUP) v = p.row_tok ? sm.idx[t] : sm.idx[t] / p.topk;
    else v = p.row_pos ? sm.idx[t] : m0 + t;
    return (v >= 0 && v < p.a_rows) ? v : -1;
  };
  // Output row of tile row t < mc.
  auto out_row = [&](int t) -> int64_t {
    if (!p.row_pos) return m0 + t;
    return GATEUP ? sm.pos[t] : sm.idx[t];
  };
  // Rows past the tile's end, and rows with a bad index, read the tile's last
  // row (row 0 if that one is bad too): finite codes, and results that are
  // not written (a bad row's are unspecified).
  const int a_last = max(row_index(mc - 1), 0);
  auto safe_row = [&](int t) {
    const int v = t < mc ? row_index(t) : -1;
    return v >= 0 ? v : a_last;
  };
  // Expert rows: wave w < groups loads group w, 8 rows per load, lane l the 16
  // bytes at LDS position l % 8 of row l / 8.
  uint32_t a_off[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int t = 32 * wave + 8 * i + (lane >> 3);
    a_off[i] = (uint32_t)safe_row(t) * (uint32_t)p.K + (((lane & 7) ^ ((t >> 1) & 7)) << 4);
  }
  const int loads_rows = wave < groups;
  const uint32_t lds_a = lds_address(sm.a) + wave * 4096;
  auto load_row = [&](int on, int blk, int i) {  // i = 0 .. 3
    async_load_1k_if(on, p.a + (int64_t)blk * kBlock, a_off[i], lds_a + (blk & 1) * kStageA + i * 1024);
  };
  // Row scales of K blocks 4 q .. 4 q + 3: waves 0-3, one row per lane.
  const uint32_t s_off = (uint32_t)safe_row((wave & 3) * 64 + lane) * (uint32_t)(nb * 4);
  const int loads_scales = wave < 4 && wave * 64 < mc;
  const uint32_t lds_s = lds_address(sm.sa) + wave * 1024;
  auto load_scales = [&](int on, int q) {
    async_load_1k_if(on, p.sa + kScaleWin * q, s_off, lds_s + (q & 1) * (int)sizeof(sm.sa[0]));
  };
  load_scales(loads_scales, 0);
#pragma unroll
  for (int i = 0; i < 4; ++i) load_row(loads_rows, 0, i);

  // acc[a][b][i]: weight row 8*(i/4) + 4*g2 + i%4 of operand a (GATEUP: rows
  // 0-15 gate, 16-31 up), expert row r32 of the wave's group b.
  v16f acc[2][4];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.0f;

  // LDS bytes of this lane's operand pieces (stage 0; stage 1 is 32 KB on).
  const uint8_t* wp = &sm.w[0][0] + wr * 8192 + (r32 >> 4) * 2048 + packed_lane_offset(0, 2 * g2, r32 & 15);
  const uint8_t* ap[2][2];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int q = 0; q < 2; ++q) ap[h][q] = &sm.a[0][0] + grp0 * 4096 + swz(r32, 4 * h + 2 * g2 + q);
  const float* sap = &sm.sa[0][grp0 * 32 + r32][0];

  // The K loop of a wave with NQ groups.  Two barriers a step, W(j) = weights
  // of K block j, A(j) = expert rows:
  //   ready(j)  W(j) and A(j) have landed for every wave, and every wave has
  //             read A(j - 1), whose stage takes A(j + 1) from here on;
  //   taken(j)  every wave has W(j) in registers: its stage takes W(j + 2).
  // ready(j + 1) stands inside the last group of step j: the step's operands
  // of the first K half are dead by then, so the next step's are read under
  // the remaining MFMAs, and no wave starts a step by waiting for LDS.  Loads
  // go out between MFMAs: a wave issues in order, and eight waves' loads queue
  // for the address unit.
  auto k_loop = [&](auto nq_tag) {
    constexpr int NQ = decltype(nq_tag)::value;
    constexpr int NL = NQ > 0 ? NQ : 1;
    // Weight operands [a][K half]; expert-row operand of the first K half (two,
    // by group: read three MFMAs ahead, an LDS read takes longer than two) and
    // of the second.
    v8i wa[2][2], x0[2], x1;
    float sa[NL], sw0, sw1;
    v16f d0 = v16f{}, d1 = v16f{};
    float s0 = 0.0f, s1 = 0.0f;  // scales of d1 (pending over the step's end)
    auto promote = [&](v16f& c, const v16f& d) {
#pragma unroll
      for (int i = 0; i < 8; ++i) c[i] += d[i] * s0;
#pragma unroll
      for (int i = 8; i < 16; ++i) c[i] += d[i] * s1;
    };
    auto x_operand = [&](int h, int b, int st) {
      return join_v8i(*reinterpret_cast<const uint4*>(ap[h][0] + st * kStageA + b * 4096),
                      *reinterpret_cast<const uint4*>(ap[h][1] + st * kStageA + b * 4096));
    };
    auto read_step = [&](int h, int j) {  // K half h of step j's operands (and, with the second, its scales)
      const int st = j & 1;
#pragma unroll
      for (int a = 0; a < 2; ++a)
        wa[a][h] = join_v8i(*reinterpret_cast<const uint4*>(wp + st * kStageW + a * 4096 + h * 1024),
                            *reinterpret_cast<const uint4*>(wp + st * kStageW + a * 4096 + h * 1024 + 512));
      if (h == 0) x0[0] = x_operand(0, 0, st);
      else x1 = x_operand(1, 0, st);
      if (h == 1) {
        const float* sj = sap + ((j / kScaleWin) & 1) * (kPrefillWideRows * kScaleWin) + (j & (kScaleWin - 1));
#pragma unroll
        for (int b = 0; b < NQ; ++b) sa[b] = sj[b * 32 * kScaleWin];
        const int js = min(j, kWideMaxBlocks - 1);
        sw0 = sm.sw[GATEUP ? 0 : wr >> 1][js];
        sw1 = GATEUP ? sm.sw[1][js] : sw0;
      }
    };
    auto fence = [&]() { __builtin_amdgcn_sched_barrier(0); };
    // ready(j + 1) in step j: the newest loads are W(j + 2), if there is one.
    auto ready = [&](int j) {
      asm volatile("s_cmp_lt_i32 %0, %1\n\ts_cbranch_scc0 .Lmoe_all_%=\n\t"
                   "s_waitcnt vmcnt(4) lgkmcnt(0)\n\ts_barrier\n\ts_branch .Lmoe_go_%=\n"
                   ".Lmoe_all_%=:\n\ts_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier\n.Lmoe_go_%=:"
                   :
                   : "s"(j + 2), "s"(nb)
                   : "memory", "scc");
      fence();
    };
    auto taken = [&]() {
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      fence();
    };
    wait_async_and_barrier<0>();  // ready(0)
    if (NQ > 0) {
      read_step(0, 0);
      read_step(1, 0);
    }
    for (int j = 0; j < nb; ++j) {
      const int st = j & 1;
      const int do_scales = loads_scales & ((j & (kScaleWin - 1)) == 0) & (j + kScaleWin < nb);
      const int do_rows = loads_rows & (j + 1 < nb), do_weights = j + 2 < nb;
      auto load_slot = [&](int i) {
        if (i == 0) load_scales(do_scales, j / kScaleWin + 1);
        if (i < 4) load_row(do_rows, j + 1, i);
        else if (i < 8) load_weight(do_weights, j + 2, i - 4);
        fence();
      };
      if (NQ == 0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) load_slot(i);
        taken();
#pragma unroll
        for (int i = 4; i < 8; ++i) load_slot(i);
        ready(j);
      }
#pragma unroll
      for (int b = 0; b < NQ; ++b) {
        const bool last = b + 1 == NQ;
        d0 = mfma_f8_32x32x64(wa[0][0], x0[b & 1], v16f{});
        if (!last) x0[(b + 1) & 1] = x_operand(0, b + 1, st);
        promote(acc[1][b > 0 ? b - 1 : NL - 1], d1);
        load_slot(4 * b);
        if (b > 0) load_slot(4 * b + 1);
        d1 = mfma_f8_32x32x64(wa[1][0], x0[b & 1], v16f{});
        load_slot(b > 0 ? 4 * b + 2 : 1);
        if (b > 0) load_slot(4 * b + 3);  // all of W(j + 2) goes out before ready(j + 1), which counts on it
        if (NQ == 1) {
          load_slot(2);
          load_slot(3);
          taken();
#pragma unroll
          for (int i = 4; i < 8; ++i) load_slot(i);
        }
        if (last) {
          ready(j);
          read_step(0, j + 1);
        }
        fence();
        d0 = mfma_f8_32x32x64(wa[0][1], x1, d0);
        fence();
        if (b == 0 && NQ > 1) {
          load_slot(2);
          load_slot(3);
          taken();
        }
        d1 = mfma_f8_32x32x64(wa[1][1], x1, d1);
        s0 = sa[b] * sw0;
        s1 = GATEUP ? sa[b] * sw1 : s0;
        fence();
        if (last) read_step(1, j + 1);
        else x1 = x_operand(1, b + 1, st);
        fence();
        promote(acc[0][b], d0);
        fence();
      }
    }
    if (NQ > 0) promote(acc[1][NL - 1], d1);
  };
  switch (nq) {
    case 0: k_loop(std::integral_constant<int, 0>{}); break;
    case 1: k_loop(std::integral_constant<int, 1>{}); break;
    case 2: k_loop(std::integral_constant<int, 2>{}); break;
    case 3: k_loop(std::integral_constant<int, 3>{}); break;
    default: k_loop(std::integral_constant<int, 4>{}); break;
  }

  if (!GATEUP) {
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int t = (grp0 + b) * 32 + r32;
      if (b < nq && t < mc) {
        float* dst = p.y + out_row(t) * p.N + nt * kPrefillWeightRows + wr * 64 + g2 * 4;
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            *reinterpret_cast<v4f*>(dst + a * 32 + q * 8) =
                v4f{acc[a][b][4 * q], acc[a][b][4 * q + 1], acc[a][b][4 * q + 2], acc[a][b][4 * q + 3]};
      }
    }
  } else {
    // h = SiLU(G) * U for channels 16 (2 wr + a) + 8*(i/4) + 4*g2 + i%4 (i < 8)
    // of the wave's rows; per-row amax over the lane's 16 channels, the other
    // K-half lane (g2) and the four weight-row quarters.
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      float mx = 0.0f;
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          acc[a][b][i] = silu_mul_fast(acc[a][b][i], acc[a][b][i + 8]);
          mx = fmaxf(mx, fabsf(acc[a][b][i]));
        }
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      if (g2 == 0 && b < nq) sm.rowmax[wr][(grp0 + b) * 32 + r32] = mx;
    }
    __syncthreads();
    uint8_t* qtile = &sm.a[0][0];  // [256][128] swizzled, the K-loop buffers are free now
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int t = (grp0 + b) * 32 + r32;
      if (b < nq) {
        const float amax = fmaxf(fmaxf(sm.rowmax[0][t], sm.rowmax[1][t]), fmaxf(sm.rowmax[2][t], sm.rowmax[3][t]));
        const float s = amax / kE4M3Max;
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
          for (int half = 0; half < 2; ++half)
            *reinterpret_cast<uint32_t*>(qtile + swz(t, 2 * wr + a) + 8 * half + 4 * g2) =
                quantize4_e4m3(acc[a][b][4 * half], acc[a][b][4 * half + 1], acc[a][b][4 * half + 2],
                               acc[a][b][4 * half + 3], s);
        if (wr == 0 && g2 == 0 && t < mc) p.sh[out_row(t) * (p.N / kBlock) + nt] = s;
      }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int c = tid + i * kThreads;
      const int row = c >> 3, col = (c & 7) * 16;
      if (row < mc)
        *reinterpret_cast<uint4*>(p.qh + out_row(row) * p.N + nt * kBlock + col) =
            *reinterpret_cast<const uint4*>(qtile + swz(row, c & 7));
    }
  }
}

// Work items (expert m-tile, n-tile) in the order of tile_of, in eight equal
// ranges, one per XCD, each a queue: a workgroup takes the next item of its own
// XCD's range and, once that is empty, of the other ranges in turn.  The ranges
// keep an expert's items on one XCD's L2; the queues even out ranges of unequal
// tiles (under skewed routing a range of full tiles takes several times as long
// as a range of experts with a few rows).  Wave 0 asks for the next item before
// its tile and waits for the answer (one round trip, two or more once its own
// range is empty), the other waves at the tile's first barrier; only the
// hand-over through LDS is behind the tile.  A queue's counter only grows, so every workgroup ends: one that
// finds nothing stops (another may still be taking the last items).
typedef const __attribute__((address_space(4))) PrefillArgs KernArg;

template <bool GATEUP>
__global__ __launch_bounds__(kThreads) void ffn_prefill_wide_kernel(PrefillArgs p) {
  __shared__ __attribute__((aligned(1024))) Smem sm;
  int total = p.mtile_start[p.n_units];
  if (total > p.max_mtiles) total = (int)p.max_mtiles;  // inconsistent offsets: only described m-tiles run
  const int real = total * p.n_tiles;                   // < 2^31 (the grid bound is checked on the host)
  const int per = (real + kXcd - 1) / kXcd;
  int32_t* const counters = p.queue + (GATEUP ? 0 : kXcd);
  const int home = blockIdx.x % kXcd, team = gridDim.x / kXcd;  // the grid is a multiple of kXcd
  // A workgroup's first item is its place in its range; the counters count the
  // items taken after the first `team` ones.
  auto at = [&](int x, int i) { return i < per && x * per + i < real ? x * per + i : -1; };
  bool home_left = true;
  auto take = [&]() {  // thread 0: the next item, or -1
    if (home_left) {
      const int item = at(home, team + atomicAdd(counters + home, 1));
      if (item >= 0) return item;
      home_left = false;
    }
    // The other ranges' counters in one round trip; only those that have
    // items left are asked (an add per empty range and workgroup took 25 us
    // at the end of every launch).
    int seen[kXcd];
#pragma unroll
    for (int d = 1; d < kXcd; ++d)
      seen[d] = __hip_atomic_load(counters + (home + d) % kXcd, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
    for (int d = 1; d < kXcd; ++d) {
      const int x = (home + d) % kXcd;
      if (at(x, team + seen[d]) < 0) continue;
      const int item = at(x, team + atomicAdd(counters + x, 1));
      if (item >= 0) return item;
    }
    return -1;
  };
  if (threadIdx.x == 0) sm.next = at(home, blockIdx.x / kXcd);
  for (;;) {
    __syncthreads();  // sm.next is written, and the last tile's LDS is free
    const int item = __builtin_amdgcn_readfirstlane(sm.next);
    if (item < 0) return;
    __syncthreads();  // sm.next is read
    int next = -1;
    if (threadIdx.x == 0) next = take();
    // The tile's values depend on these two as far as the compiler knows, so
    // that it forms them anew for every tile: kept in registers over the K loop
    // (64 of them) they were spilled, and the loop with them.
    KernArg* args = (KernArg*)__builtin_amdgcn_kernarg_segment_ptr();
    int tid = threadIdx.x;
    asm volatile("" : "+s"(args), "+v"(tid));
    wide_tile<GATEUP>(*(const PrefillArgs*)args, sm, item, tid);
    if (threadIdx.x == 0) sm.next = next;
  }
}

}  // namespace

// Expected cost of a launch pair with t-row tiles, in units of a 32-row group's
// K step: per GEMM the rounds of tiles over the CUs (whole rounds while there
// are few, since one more round is then a large part; a queue's tail of half a
// round beyond) times a tile's groups and its fixed part (0.75 groups), times K.
// An expert's tiles are those of the mean row count, averaged over one standard
// deviation of a uniform draw around it.
static double tile_cost(const moe_dims_t& d, double mean_rows, double n_units, int t) {
  const double spread = sqrt(mean_rows);
  const double tiles = 0.5 * (std::max(1.0, ceil((mean_rows - spread) / t)) + ceil((mean_rows + spread) / t));
  const double per_tile = (mean_rows / 32 + 0.5) / tiles + 0.75;
  auto rounds = [&](int n_tiles) {
    const double r = n_units * tiles * n_tiles / kWideWorkgroups;
    return r <= 3.0 ? ceil(r) : r + 0.5;
  };
  return per_tile * (rounds(d.inter / kBlock) * d.hidden + rounds(d.hidden / kPrefillWeightRows) * d.inter);
}

// Wide tiles where they are expected to be faster by that cost, from about 120
// rows per expert, where the narrow tiles start to need a second tile per
// expert (below, both have one tile per expert and the narrow kernel is 2 - 3 %
// faster: 3072 tokens, 96 rows per expert: 1349 against 1405, 830 against 847
// us), and where a CU gets kWideMinRounds full tiles or more (of both GEMMs,
// weighted by their K).  The cost knows the mean row count only; with few tiles
// per CU one more tile decides, and skewed routing brings it: whole layers, wide
// against narrow, uniform | Zipf(0.5) | Zipf(1):
//   H 4096, I 1536, 16 experts,  2046 rows, 0.4 rounds: 0.78 | 1.07 | 1.06
//   H 4096, I 4096,  8 experts,  3500 rows, 1.3:        0.96 | 1.26 | 1.30
//   H 4096, I 2048, 32 experts,  4092 rows, 1.0:        0.94 | 1.28 | 1.28
//   H 3072, I 1536, 64 experts,  9000 rows, 1.6:        0.87 | 1.04 | 1.07
//   H 7168, I 2048, 64 experts,  8184 rows, 2.3:        0.93 | 1.06 | 1.01
//   H 4096, I 1024, 128 experts, 16384 rows, 2.4:       0.93 | 1.00 | 0.99
//   H 4096, I 2048, 32 experts, 12000 rows, 2.9:        0.93 | 0.96 | 0.97
//   H 7168, I 2048, 64 experts, 16384 rows, 4.7:        0.91 | 0.91 | 0.97
// Over 19 shapes, 4 to 256 experts, 30 to 1400 rows per expert, the cost alone took
// wide tiles where they had up to 1.33 times the narrow ones' time; with the rounds
// none has more than 1.03.
// Shapes: row scales come four K blocks at a time (K a multiple of 512, sx
// 16-byte aligned), 32-bit row offsets, and enough rows that the tile table,
// sized for 128-row tiles, has room for the queue counters (about 1024).
int prefill_tile_rows(const moe_dims_t& d, const PrefillRows& r, const float* sx) {
  const int step = kBlock * kScaleWin, kmax = kWideMaxBlocks * kBlock;
  if (d.hidden % step || d.inter % step || d.hidden > kmax || d.inter > kmax || !aligned(sx, 16) ||
      (int64_t)r.tokens * d.hidden > 0xffffffffll || r.rows * d.inter > 0xffffffffll || r.unit_rows < r.n_units)
    return kPrefillTileRows;
  const int64_t wide_tiles = (r.rows + kPrefillWideRows - 1) / kPrefillWideRows + std::min<int64_t>(r.rows, r.n_units);
  if (wide_tiles + kQueueDescs > r.max_mtiles) return kPrefillTileRows;
  const double full = (double)r.unit_rows / (kPrefillWideRows * kWideWorkgroups);
  const double rounds = full * (d.inter / kBlock * (double)d.hidden + d.hidden / kPrefillWeightRows * (double)d.inter) /
                        ((double)d.hidden + d.inter);
  if (rounds < kWideMinRounds) return kPrefillTileRows;
  const double mean = (double)r.unit_rows / r.n_units;
  return tile_cost(d, mean, r.n_units, kPrefillWideRows) < 0.99 * tile_cost(d, mean, r.n_units, kPrefillTileRows)
             ? kPrefillWideRows
             : kPrefillTileRows;
}

moe_status_t launch_prefill_wide(bool gateup, const PrefillArgs& a, int64_t max_mtiles, hipStream_t stream) {
  if (max_mtiles * a.n_tiles > 0x7fffffff) return fail(MOE_ERR_UNSUPPORTED_SHAPE, "ffn_prefill: grid too large");
  const int64_t grid = std::min<int64_t>((max_mtiles * a.n_tiles + kXcd - 1) / kXcd * kXcd, kWideWorkgroups);
  if (gateup)
    MOE_LAUNCH("ffn_prefill_gateup", ffn_prefill_wide_kernel<true>, dim3((unsigned)grid), dim3(kThreads), 0, stream, a);
  else
    MOE_LAUNCH("ffn_prefill_down", ffn_prefill_wide_kernel<false>, dim3((unsigned)grid), dim3(kThreads), 0, stream, a);
  return check_launch(gateup ? "ffn_prefill_gateup" : "ffn_prefill_down");
}

}  // namespace moe
