// Shared by the prefill GEMM kernels (ffn_prefill.hip, ffn_prefill_wide.hip):
// arguments, work items, the LDS swizzle and the MFMA.
#pragma once

#include "common.h"

namespace moe {

typedef float v16f __attribute__((ext_vector_type(16)));

constexpr int kPrefillWeightRows = 256;  // weight rows per tile
constexpr int kBandRows = 1024;          // expert rows per band of the work-item order (see tile_of)

struct PrefillArgs {
  const uint8_t* a;           // e4m3 activations [a_rows, K]
  const float* sa;            // [a_rows, K/128]
  const int32_t* sorted_src;  // GATEUP without row tables: A row of sorted row p = sorted_src[p] / topk; else unused
  const int32_t* row_pos;     // NULL: tile rows are sorted positions; else the sorted position of launch row v
  const int32_t* row_tok;     // GATEUP with row_pos: the token (A row) of launch row v
  int topk;
  int a_rows;
  const int32_t* mtile_start; // [n_units+1] exclusive scan of the experts' m-tile counts
  const int4* desc;           // [max_mtiles] m-tile block descriptors (prefill_tiles_kernel)
  int64_t max_mtiles;         // bound on the m-tiles (sizes desc)
  int32_t* queue;             // wide tiles: two sets of kXcd work-queue counters (gate/up, down), zeroed with the table; else NULL
  int tile_rows;              // expert rows per m-tile at most (kPrefillTileRows or kPrefillWideRows)
  int n_units;                // experts of the launch
  const uint8_t* w0;          // GATEUP: W_gate [E, N, K]; DOWN: W_down [E, N, K]; packed tiles
  const float* s0;
  const uint8_t* w1;          // GATEUP: W_up, packed tiles
  const float* s1;
  int N, K;                   // N: output columns of the expert (I for gate/up, H for down)
  int n_tiles;                // GATEUP: N/128; DOWN: N/256
  float* y;                   // DOWN output fp32 [rows, N]
  uint8_t* qh;                // GATEUP output e4m3 [rows, N]
  float* sh;                  // GATEUP output [rows, N/128]
};

// LDS byte offset of 16-byte chunk c (0..7) of row `row` in a 128-byte-row
// tile.  gfx950's LDS serves 256 bytes per clock (64 four-byte banks), so
// two consecutive 128-byte rows share one bank row; the chunk index is
// XOR-ed with (row / 2) % 8, so the 16 rows that a quarter-wave b128 read
// touches fill all 16 sixteen-byte bank slots (measured on gfx950: about
// 195 B/clk per CU this way, 122 with the chunk XOR-ed by row % 8, whose
// rows r and r + 8 collide, and 32 unswizzled).
__device__ __forceinline__ int swz(int row, int c) { return row * kBlock + ((c ^ ((row >> 1) & 7)) << 4); }

__device__ __forceinline__ v16f mfma_f8_32x32x64(const v8i& a, const v8i& b, const v16f& c) {
  // Scale operands 0: the compiler emits the unscaled v_mfma_f32_32x32x64_f8f6f4
  // (e4m3 operands, no block scales; see mfma_f8_16x16x128).
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 0, 0, 0, 0, 0, 0);
}

// The tile of work item `item`: expert u owns items [mtile_start[u],
// mtile_start[u+1]) * n_tiles, in bands of B = kBandRows / tile_rows
// consecutive m-tiles, each band n-tile major: item = mtile_start[u] *
// n_tiles + B * n_tiles * band + nt * width + (mt - B * band) (width = the band's m-tiles; an
// expert with at most B m-tiles is one band).  The m-tiles that read the
// same weight slice (same nt) are neighbours, so they run together on one
// XCD and the slice comes from HBM once per band (m-tile major order
// fetched the weights once per m-tile); and an expert with many m-tiles
// re-reads its token rows once per band pass instead of once per n-tile
// (one n-tile-major pass over 141 m-tiles evicts them from L2 before the
// next n-tile reads them again).  The expert's ceil(M/32) row groups are dealt evenly over its
// mcount tiles (tile mt gets q/mcount groups, one more for mt < q % mcount):
// the same MFMA work as full tiles plus a tail, but tiles of similar size,
// which advance through their shared weight slice at similar speed, so the
// slice is fetched from HBM once and read by the others from L2 (a 1-32-row
// tail tile ran about 3.6 times faster than the full tiles and fetched the
// slice ahead of them; gate/up read 1.7 times its algorithmic bytes).
struct Tile {
  int e, m0, mc, nt;  // expert, first row (a sorted position, or a launch row with row tables), rows, n-tile
};

__device__ __forceinline__ Tile tile_of(const PrefillArgs& p, int item) {
  const int4 d = p.desc[item / p.n_tiles];
  const int e = d.x, s0 = d.y, o0 = d.z, o1 = d.w;
  const int mcount = (o1 - o0 + p.tile_rows - 1) / p.tile_rows;
  const int local = item - s0 * p.n_tiles;
  const int kband = kBandRows / p.tile_rows;  // m-tiles per band
  const int band = local / (kband * p.n_tiles);
  const int bw = min(kband, mcount - band * kband);
  const int in_band = local - band * kband * p.n_tiles;
  const int ntx = in_band / bw;
  const int mt = band * kband + (in_band - ntx * bw);
  const int q = (o1 - o0 + 31) >> 5;
  const int base = q / mcount, extra = q - base * mcount;
  const int first = o0 + 32 * (mt * base + min(mt, extra));
  const int groups = base + (mt < extra ? 1 : 0);
  return Tile{e, first, min(32 * groups, o1 - first), ntx};
}


// The work item of this workgroup, or -1: XCD-major over the real items (the
// grid is an upper bound): XCD x takes items [x*per, (x+1)*per) in order.
__device__ __forceinline__ int prefill_item(const PrefillArgs& p) {
  int total = p.mtile_start[p.n_units];
  if (total > p.max_mtiles) total = (int)p.max_mtiles;  // inconsistent offsets: only described m-tiles run
  const int real = total * p.n_tiles;                   // < 2^31 (the grid bound is checked on the host)
  const int per = (real + kXcd - 1) / kXcd;
  const int slot = blockIdx.x / kXcd;
  if (slot >= per) return -1;
  const int item = (int)(blockIdx.x % kXcd) * per + slot;
  return item < real ? item : -1;
}

// The tile rows of a launch over r, activation scales at sx (see
// ffn_prefill_wide.hip).
int prefill_tile_rows(const moe_dims_t& d, const PrefillRows& r, const float* sx);
moe_status_t launch_prefill_wide(bool gateup, const PrefillArgs& a, int64_t max_mtiles, hipStream_t stream);

}  // namespace moe
