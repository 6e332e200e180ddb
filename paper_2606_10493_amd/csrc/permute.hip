// Token -> expert permutation: a stable counting sort of the flat slots
// f = t*k + j by expert id (tokens gated and sorted by expert into per-expert
// token lists, as in the standard expert-parallel workflow of the paper).
//
// A token lists each expert at most once, so within one expert the stable
// order by f is the order by token.  Each 256-token chunk therefore builds,
// in LDS, one 256-bit token mask per expert (4 x 64-bit words, set with an
// order-independent atomic OR).  The rank of (t, e) inside the chunk is the
// number of set bits below t in e's mask, so the scatter is exact and
// deterministic without any order-dependent atomics.
//
// Slots whose id is out of range, or repeats an earlier slot's id in the
// same token, are reported in the device status word and parked after all
// valid rows (positions expert_offsets[E] .. T*k-1, in slot order), so the
// outputs stay a bijection and every later index stays in bounds.  The atomic
// OR returns the word before it: a bit that was set already is a repeated id
// (how many there are does not depend on the order of the atomics; which slot
// of the two is the earlier one is only looked up when there are any).
//
// These kernels are latency chains of a few microseconds (launch, one load
// round trip, LDS, scan), so a chunk has 1024 threads, each holding its at
// most 8 slot ids in registers, and as little as possible is a launch of its
// own:
//   one chunk  (T <= 256): permute_small_kernel does count, scan and scatter
//              (layer_prologue_kernel: the same, beside the activation quantization).
//   several chunks: permute_count_kernel (layer: beside the activation
//              quantization, quant_count_kernel) -> permute_scatter_kernel,
//              whose workgroups each sum the chunks' counts again.  Beyond
//              kMaxFusedScan chunks that re-reading grows with the square of
//              the chunks and a scan of its own goes first (512 chunks, the
//              sort in all: 256 experts 35 us, 1024 experts 95 us; 547 chunks
//              with the scan, 256 experts 103 us).
// In a layer call of the prefill regime the kernel that knows the experts'
// counts also writes the m-tile table of the GEMMs (TilesOut), with more than
// kTinySlots slots and up to kMaxFusedScan chunks; else prefill_tiles_kernel does.
//
// Measured (rocprofv3, one layer's quantization, sort and m-tile table): 201
// tokens x 8 slots over 256 experts 19.2 us in two launches -> 5.6 us in one;
// 509 tokens over 128 experts 31.0 us in five launches -> 11.3 us in two;
// 8192 tokens 70.2 us -> 53.3 us (45.0 of it the quantization, HBM bound).
// 256-thread chunks whose threads walked a token's k slots one after the
// other took 8.6 us to count and 11.2 us to scatter; these take 4.8 and 6.5.
#include "common.h"

namespace moe {

namespace {

constexpr int kChunk = 256;         // tokens per workgroup
constexpr int kSortThreads = 1024;  // threads per chunk (and one per expert in the scan)
constexpr int kMaxExperts = 1024;
constexpr int kMaxTopk = 32;
constexpr int kSlotsPerThread = kChunk * kMaxTopk / kSortThreads;
constexpr int kMaxFusedScan = 512;  // chunks up to which every scatter workgroup sums all counts itself

// LDS of one chunk.
struct ChunkMasks {
  unsigned long long mask[kMaxExperts * 4];  // per expert, the chunk's tokens that list it
  int base[kMaxExperts];                     // first sorted position of the chunk's rows of each expert
  int wave_tot[kSortThreads / 64];
  int bad_count;                             // invalid slots of the chunk
};

// Token (chunk-local) of slot f < kChunk * kMaxTopk: f / k by the reciprocal.
// (f + 0.5) / k is at least 0.5 / 32 away from an integer and the product's
// error is below 8192 * 2^-22, so the truncation is exact.
__device__ __forceinline__ int token_of(int f, float inv_k) { return (int)(((float)f + 0.5f) * inv_k); }

// Clear the masks, read this thread's slots of the chunk (ids: the chunk's
// first slot, n slots) and set their mask bits; returns the thread's MOE_DEV_*
// bits.  The masks and bad_count are complete on return.
__device__ __forceinline__ uint32_t mark_slots(ChunkMasks& cm, const int32_t* __restrict__ ids, int n, float inv_k,
                                               int E, int (&id)[kSlotsPerThread]) {
  const int tid = threadIdx.x;
#pragma unroll
  for (int q = 0; q < kSlotsPerThread; ++q)
    if (q * kSortThreads < n) id[q] = ids[min(q * kSortThreads + tid, n - 1)];
  for (int i = tid; i < E * 4; i += kSortThreads) cm.mask[i] = 0ull;
  if (tid == 0) cm.bad_count = 0;
  __syncthreads();
  uint32_t err = 0;
#pragma unroll
  for (int q = 0; q < kSlotsPerThread; ++q) {
    if (q * kSortThreads >= n) break;
    const int f = q * kSortThreads + tid;
    if (f < n) {
      uint32_t bad = MOE_DEV_BAD_EXPERT_ID;
      if (id[q] >= 0 && id[q] < E) {
        const int t = token_of(f, inv_k);
        const unsigned long long bit = 1ull << (t & 63);
        bad = (atomicOr(&cm.mask[id[q] * 4 + (t >> 6)], bit) & bit) ? MOE_DEV_DUP_EXPERT_ID : 0u;
      }
      if (bad) {
        err |= bad;
        atomicAdd(&cm.bad_count, 1);
      }
    }
  }
  __syncthreads();
  return err;
}

// Whether slot f (chunk-local) is valid: its id is in range and no earlier
// slot of its token has the same id.  Only chunks with invalid slots ask.
__device__ __forceinline__ bool slot_valid(const int32_t* __restrict__ ids, int f, int k, int E) {
  const int id = ids[f];
  bool ok = id >= 0 && id < E;
#pragma unroll 1
  for (int i = f - f % k; i < f; ++i) ok &= ids[i] != id;
  return ok;
}

// Rank of token lt (chunk-local) among the chunk's tokens routed to e.
__device__ __forceinline__ int rank_of(const unsigned long long* mask, int e, int lt) {
  const int word = lt >> 6;
  const unsigned long long below = (1ull << (lt & 63)) - 1ull;
  int r = __popcll(mask[e * 4 + word] & below);
  for (int w = 0; w < word; ++w) r += __popcll(mask[e * 4 + w]);
  return r;
}

__device__ __forceinline__ int mask_count(const unsigned long long* mask, int e) {
  return __popcll(mask[e * 4]) + __popcll(mask[e * 4 + 1]) + __popcll(mask[e * 4 + 2]) + __popcll(mask[e * 4 + 3]);
}

__device__ __forceinline__ void report(int32_t* dev_status, uint32_t err) {
  // Any-lane OR, then one atomic per wave.
  for (int m = 32; m >= 1; m >>= 1) err |= (uint32_t)__shfl_xor((int)err, m, 64);
  if (dev_status && err && (threadIdx.x & 63) == 0) atomicOr(dev_status, (int)err);
}

// The chunk's slots (chunk-local f -> flat slot f0 + f) to their positions:
// valid ones to base[e] + rank, invalid ones in slot order from bad_base (their
// numbers by a scan over each kSortThreads slots: 256 tokens x 8 slots, half of
// them bad, 8.5 us, x 32 slots 38 us; one thread that walked the chunk's slots
// took 0.48 and 5.6 ms).
__device__ __forceinline__ void scatter_slots(ChunkMasks& cm, const int32_t* __restrict__ ids, int n, int k,
                                              float inv_k, int E, const int (&id)[kSlotsPerThread], int32_t f0,
                                              int32_t bad_base, int32_t* __restrict__ sorted_src,
                                              int32_t* __restrict__ dest_row) {
  const int tid = threadIdx.x;
  if (cm.bad_count == 0) {
#pragma unroll
    for (int q = 0; q < kSlotsPerThread; ++q) {
      if (q * kSortThreads >= n) break;
      const int f = q * kSortThreads + tid;
      if (f < n) {
        const int32_t p = cm.base[id[q]] + rank_of(cm.mask, id[q], token_of(f, inv_k));
        dest_row[f0 + f] = p;
        sorted_src[p] = f0 + f;
      }
    }
    return;
  }
  for (int q0 = 0; q0 < n; q0 += kSortThreads) {
    const int f = q0 + tid;
    const bool ok = f < n && slot_valid(ids, f, k, E);
    int bad;
    int32_t p = bad_base + block_exclusive_scan(f < n && !ok, cm.wave_tot, &bad);
    bad_base += bad;
    if (ok) p = cm.base[ids[f]] + rank_of(cm.mask, ids[f], token_of(f, inv_k));
    if (f < n) {
      dest_row[f0 + f] = p;
      sorted_src[p] = f0 + f;
    }
  }
}

// The expert offsets and, if asked for, the m-tile table (the same as
// prefill_tiles_kernel writes for one chunk of rows), from expert
// threadIdx.x's first row and row count.
__device__ __forceinline__ void write_offsets(ChunkMasks& cm, int E, int first, int count, int total_valid,
                                              int32_t* __restrict__ offsets, const TilesOut& tiles) {
  const int e = threadIdx.x;
  if (e < E) offsets[e] = first;
  if (e == 0) offsets[E] = total_valid;
  if (!tiles.mtile_start) return;
  const int cnt = e < E ? (count + tiles.tile_rows - 1) / tiles.tile_rows : 0;
  int total;
  const int excl = block_exclusive_scan(cnt, cm.wave_tot, &total);
  if (e < E) {
    tiles.mtile_start[e] = excl;
    for (int b = excl; b < excl + cnt && b < tiles.max_mtiles; ++b)
      tiles.desc[b] = make_int4(e, excl, first, first + count);
  }
  if (e == 0) tiles.mtile_start[E] = total;
  if (tiles.queue && e < kQueueInts) tiles.queue[e] = 0;
}

// One chunk (T <= 256): mask, scan and scatter in one workgroup.
__device__ __forceinline__ void permute_one_chunk(const int32_t* __restrict__ ids, int T, int k, int E,
                                                  int32_t* __restrict__ offsets, int32_t* __restrict__ sorted_src,
                                                  int32_t* __restrict__ dest_row, int32_t* __restrict__ dev_status,
                                                  const TilesOut& tiles) {
  __shared__ ChunkMasks cm;
  const float inv_k = 1.0f / (float)k;
  int id[kSlotsPerThread];
  const uint32_t err = mark_slots(cm, ids, T * k, inv_k, E, id);
  const int e = threadIdx.x;
  const int count = e < E ? mask_count(cm.mask, e) : 0;
  int total_valid;
  const int first = block_exclusive_scan(count, cm.wave_tot, &total_valid);
  if (e < E) cm.base[e] = first;
  __syncthreads();
  scatter_slots(cm, ids, T * k, k, inv_k, E, id, 0, total_valid, sorted_src, dest_row);
  write_offsets(cm, E, first, count, total_valid, offsets, tiles);
  report(dev_status, err);
}

// At most kTinySlots slots (decode batches): the same results as
// permute_one_chunk with two barriers and no loop whose trip count depends
// on the slot count.  Each slot gets a key: its id if valid, INT_MAX if not
// (or past the slots).  Slot f's stable position among the valid slots is the
// number of keys g with (key[g], g) < (key[f], f); an invalid slot goes after
// all valid ones, in slot order (a ballot prefix count); offsets[e] is the
// number of keys below e.  The counts read the 64 keys as 16 broadcast int4
// LDS loads, issued together.
constexpr int kTinySlots = 64;

__device__ __forceinline__ void permute_tiny(const int32_t* __restrict__ ids, int T, int k, int E,
                                             int32_t* __restrict__ offsets, int32_t* __restrict__ sorted_src,
                                             int32_t* __restrict__ dest_row, int32_t* __restrict__ dev_status) {
  __shared__ int sid[kTinySlots];
  __shared__ __attribute__((aligned(16))) int key[kTinySlots];
  const int n = T * k, tid = threadIdx.x;
  if (tid < kTinySlots) {
    int id = -1;
    if (tid < n) {
      const int32_t v = ids[tid];
      id = (v >= 0 && v < E) ? v : -1;
    }
    sid[tid] = id;
  }
  __syncthreads();
  uint32_t err = 0;
  bool valid = false;
  int me = INT_MAX;
  if (tid < n) {
    const int t = tid / k, j = tid - t * k;
    const int id = sid[tid];
    if (id < 0) {
      err = MOE_DEV_BAD_EXPERT_ID;
    } else {
      for (int i = 0; i < j; ++i)
        if (sid[t * k + i] == id) err = MOE_DEV_DUP_EXPERT_ID;
    }
    valid = err == 0;
    me = valid ? id : INT_MAX;
  }
  if (tid < kTinySlots) key[tid] = me;
  // Slots live in wave 0 (n <= 64): its ballots count valid and invalid slots.
  const unsigned long long vmask = __ballot(tid < n && valid);
  const unsigned long long bmask = __ballot(tid < n && !valid);
  __syncthreads();
  const int4* k4 = reinterpret_cast<const int4*>(key);
  if (tid < n) {
    int pos;
    if (valid) {
      pos = 0;
#pragma unroll
      for (int q = 0; q < kTinySlots / 4; ++q) {
        const int4 v = k4[q];
        const int g = 4 * q;
        pos += (v.x < me || (v.x == me && g < tid)) ? 1 : 0;
        pos += (v.y < me || (v.y == me && g + 1 < tid)) ? 1 : 0;
        pos += (v.z < me || (v.z == me && g + 2 < tid)) ? 1 : 0;
        pos += (v.w < me || (v.w == me && g + 3 < tid)) ? 1 : 0;
      }
    } else {
      pos = __popcll(vmask) + __popcll(bmask & ((1ull << tid) - 1ull));
    }
    dest_row[tid] = pos;
    sorted_src[pos] = tid;
  }
  for (int e = tid; e < E; e += blockDim.x) {
    int c = 0;
#pragma unroll
    for (int q = 0; q < kTinySlots / 4; ++q) {
      const int4 v = k4[q];
      c += (v.x < e ? 1 : 0) + (v.y < e ? 1 : 0) + (v.z < e ? 1 : 0) + (v.w < e ? 1 : 0);
    }
    offsets[e] = c;
  }
  if (tid == 0) offsets[E] = __popcll(vmask);
  report(dev_status, err);
}

// Up to kTinySlots slots one 256-thread workgroup, else kSortThreads threads.
template <bool TINY>
__global__ __launch_bounds__(TINY ? 256 : kSortThreads) void permute_small_kernel(
    const int32_t* __restrict__ ids, int T, int k, int E, int32_t* __restrict__ offsets,
    int32_t* __restrict__ sorted_src, int32_t* __restrict__ dest_row, int32_t* __restrict__ dev_status) {
  if constexpr (TINY) permute_tiny(ids, T, k, E, offsets, sorted_src, dest_row, dev_status);
  else permute_one_chunk(ids, T, k, E, offsets, sorted_src, dest_row, dev_status, TilesOut{});
}

// Layer prologue for one chunk of tokens (T <= 256), one launch instead of
// two: workgroup 0 sorts the slots (as permute_small_kernel); workgroups 1..
// quantize the bf16 activations, one group of 128 columns per 16 threads (as
// moe_quant_act).
template <bool TINY>
__global__ __launch_bounds__(TINY ? 256 : kSortThreads) void layer_prologue_kernel(
    const int32_t* __restrict__ ids, int T, int k, int E, int32_t* __restrict__ offsets,
    int32_t* __restrict__ sorted_src, int32_t* __restrict__ dest_row, int32_t* __restrict__ dev_status,
    const uint16_t* __restrict__ x, int64_t n_groups, int groups_per_row, uint8_t* __restrict__ qx,
    float* __restrict__ sx, TilesOut tiles) {
  if (blockIdx.x == 0) {
    if constexpr (TINY) permute_tiny(ids, T, k, E, offsets, sorted_src, dest_row, dev_status);
    else permute_one_chunk(ids, T, k, E, offsets, sorted_src, dest_row, dev_status, tiles);
    return;
  }
  const int64_t g = (int64_t)(blockIdx.x - 1) * (blockDim.x / 16) + (threadIdx.x >> 4);
  if (g >= n_groups) return;  // whole 16-lane groups leave together
  quant_row_group<uint16_t>(x, g, threadIdx.x & 15, groups_per_row, qx, sx);
}

// Slots of chunk c.
__device__ __forceinline__ int chunk_slots(int64_t c, int T, int k) {
  return (int)min((int64_t)kChunk, T - c * kChunk) * k;
}

// counts: [n_chunks][E+1]; entry E is the chunk's number of invalid slots.
__device__ __forceinline__ void count_chunk(int64_t c, const int32_t* __restrict__ ids, int T, int k, int E,
                                            int32_t* __restrict__ counts, int32_t* __restrict__ dev_status) {
  __shared__ ChunkMasks cm;
  int id[kSlotsPerThread];
  const uint32_t err = mark_slots(cm, ids + c * kChunk * k, chunk_slots(c, T, k), 1.0f / (float)k, E, id);
  int32_t* row = counts + c * (E + 1);
  for (int e = threadIdx.x; e < E; e += kSortThreads) row[e] = mask_count(cm.mask, e);
  if (threadIdx.x == 0) row[E] = cm.bad_count;
  report(dev_status, err);
}

__global__ __launch_bounds__(kSortThreads) void permute_count_kernel(const int32_t* __restrict__ ids, int T, int k,
                                                                     int E, int chunk0,
                                                                     int32_t* __restrict__ counts,
                                                                     int32_t* __restrict__ dev_status) {
  count_chunk((int64_t)chunk0 + blockIdx.x, ids, T, k, E, counts, dev_status);
}

// Layer call of several chunks: workgroups 0 .. n_chunks-1 count the slots,
// the others quantize the activations (64 groups each), in one launch.
__global__ __launch_bounds__(kSortThreads) void quant_count_kernel(const int32_t* __restrict__ ids, int T, int k,
                                                                   int E, int n_chunks, int32_t* __restrict__ counts,
                                                                   int32_t* __restrict__ dev_status,
                                                                   const uint16_t* __restrict__ x, int64_t n_groups,
                                                                   int groups_per_row, uint8_t* __restrict__ qx,
                                                                   float* __restrict__ sx) {
  if ((int)blockIdx.x < n_chunks) {
    count_chunk(blockIdx.x, ids, T, k, E, counts, dev_status);
    return;
  }
  const int64_t g = (int64_t)(blockIdx.x - n_chunks) * (kSortThreads / 16) + (threadIdx.x >> 4);
  if (g >= n_groups) return;  // whole 16-lane groups leave together
  quant_row_group<uint16_t>(x, g, threadIdx.x & 15, groups_per_row, qx, sx);
}

// One workgroup of 1024 threads; thread e scans expert e over the chunks.
__global__ __launch_bounds__(1024) void permute_scan_kernel(const int32_t* __restrict__ counts, int n_chunks, int E,
                                                            int32_t* __restrict__ base,
                                                            int32_t* __restrict__ offsets) {
  __shared__ int wave_tot[16];
  const int e = threadIdx.x;
  int tot = 0;
  // Unrolled by 8 so that eight independent loads go out before the first
  // wait (a plain loop waited for every chunk's count in turn).
  if (e < E) {
#pragma unroll 8
    for (int c = 0; c < n_chunks; ++c) tot += counts[(int64_t)c * (E + 1) + e];
  }
  int total_valid;
  const int excl = block_exclusive_scan(tot, wave_tot, &total_valid);
  if (e < E) {
    int run = excl;
    offsets[e] = run;
#pragma unroll 8
    for (int c = 0; c < n_chunks; ++c) {
      const int64_t i = (int64_t)c * (E + 1) + e;
      base[i] = run;
      run += counts[i];
    }
  }
  if (e == 0) {
    offsets[E] = total_valid;
    int run = total_valid;
    for (int c = 0; c < n_chunks; ++c) {
      const int64_t i = (int64_t)c * (E + 1) + E;
      base[i] = run;
      run += counts[i];
    }
  }
}

// Scatter, one chunk per workgroup.  base: the chunk bases of
// permute_scan_kernel, or NULL: each workgroup sums the counts itself, thread
// (part, e) those of expert e in the chunks part, part + parts, ... (all
// chunks, and those before its own), so that a few tens of chunks cost one
// round trip of loads; workgroup 0 writes the offsets and the m-tile table.
__global__ __launch_bounds__(kSortThreads) void permute_scatter_kernel(
    const int32_t* __restrict__ ids, int T, int k, int E, int chunk0, int n_chunks,
    const int32_t* __restrict__ counts, const int32_t* __restrict__ base, int32_t* __restrict__ offsets,
    int32_t* __restrict__ sorted_src, int32_t* __restrict__ dest_row, TilesOut tiles) {
  __shared__ ChunkMasks cm;
  __shared__ int part_sum[2][kSortThreads];  // [total, before this chunk]
  const int tid = threadIdx.x;
  const float inv_k = 1.0f / (float)k;
  const int64_t c = (int64_t)chunk0 + blockIdx.x;
  const int32_t f0 = (int32_t)(c * kChunk * k);
  const int n = chunk_slots(c, T, k);
  int id[kSlotsPerThread];
  mark_slots(cm, ids + f0, n, inv_k, E, id);
  int32_t bad_base = 0;
  if (base) {
    const int32_t* brow = base + c * (E + 1);
    for (int e = tid; e < E; e += kSortThreads) cm.base[e] = brow[e];
    bad_base = brow[E];
  } else {
    const int parts = kSortThreads / E;  // E <= kSortThreads
    const int part = tid / E, col = tid - part * E;
    int tot = 0, before = 0;
    if (part < parts) {
#pragma unroll 8
      for (int x = part; x < n_chunks; x += parts) {
        const int v = counts[x * (E + 1) + col];  // < kMaxFusedScan * 1025
        tot += v;
        before += x < c ? v : 0;
      }
    }
    part_sum[0][tid] = tot;
    part_sum[1][tid] = before;
    __syncthreads();
    tot = before = 0;
    if (tid < E)
      for (int p = 0; p < parts; ++p) {
        tot += part_sum[0][p * E + tid];
        before += part_sum[1][p * E + tid];
      }
    int total_valid;
    const int first = block_exclusive_scan(tot, cm.wave_tot, &total_valid);
    if (tid < E) cm.base[tid] = first + before;
    if (c == 0) write_offsets(cm, E, first, tot, total_valid, offsets, tiles);
    bad_base = total_valid;
    if (cm.bad_count > 0) {  // the invalid slots of the chunks before this one
      static_assert(kMaxFusedScan <= kSortThreads, "one chunk per thread");
      int bad;
      block_exclusive_scan(tid < c ? counts[tid * (E + 1) + E] : 0, cm.wave_tot, &bad);
      bad_base += bad;
    }
  }
  __syncthreads();
  scatter_slots(cm, ids + f0, n, k, inv_k, E, id, f0, bad_base, sorted_src, dest_row);
}

int64_t n_chunks_of(int32_t T) { return ((int64_t)T + kChunk - 1) / kChunk; }

}  // namespace

// A grid has less than 2^32 threads: chunks per launch of the sort's kernels.
constexpr int64_t kChunksPerLaunch = 1 << 21;

moe_status_t launch_count(const int32_t* topk_ids, int32_t T, int32_t k, int32_t E, int32_t* counts,
                          int32_t* dev_status, hipStream_t stream) {
  const int64_t nc = n_chunks_of(T);
  for (int64_t c0 = 0; c0 < nc; c0 += kChunksPerLaunch)
    MOE_LAUNCH("permute_count", permute_count_kernel, dim3((unsigned)min(nc - c0, kChunksPerLaunch)),
               dim3(kSortThreads), 0, stream, topk_ids, T, k, E, (int)c0, counts, dev_status);
  return check_launch("moe_permute");
}

// The chunks' counts -> positions.  counts: the first part of the permute workspace.
moe_status_t launch_scatter(const int32_t* topk_ids, int32_t T, int32_t k, int32_t E, int32_t* offsets,
                            int32_t* sorted_src, int32_t* dest_row, int32_t* counts, const TilesOut& tiles,
                            hipStream_t stream) {
  const int64_t nc = n_chunks_of(T);
  int32_t* base = nullptr;
  if (nc > kMaxFusedScan) {
    base = counts + nc * (E + 1);
    MOE_LAUNCH("permute_scan", permute_scan_kernel, dim3(1), dim3(1024), 0, stream, counts, (int)nc, E, base, offsets);
  }
  for (int64_t c0 = 0; c0 < nc; c0 += kChunksPerLaunch)
    MOE_LAUNCH("permute_scatter", permute_scatter_kernel, dim3((unsigned)min(nc - c0, kChunksPerLaunch)),
               dim3(kSortThreads), 0, stream, topk_ids, T, k, E, (int)c0, (int)nc, counts, base, offsets, sorted_src,
               dest_row, tiles);
  return check_launch("moe_permute");
}

// Whether launch_layer_prologue also writes a m-tile table it is given.
bool layer_prologue_writes_tiles(int32_t T, int32_t k) {
  return T <= kChunk ? T * k > kTinySlots : n_chunks_of(T) <= kMaxFusedScan;
}

// Quantize x [T, H] and sort the slots: one launch for T <= 256 tokens, two
// for more.  tiles: the m-tile table to write (see
// layer_prologue_writes_tiles), or empty.  perm_ws: moe_permute_workspace
// bytes.  Arguments are checked by the caller.
moe_status_t launch_layer_prologue(const uint16_t* x, int32_t T, int32_t H, const int32_t* topk_ids, int32_t k,
                                   int32_t E, uint8_t* qx, float* sx, int32_t* offsets, int32_t* sorted_src,
                                   int32_t* dest_row, int32_t* dev_status, const TilesOut& tiles, void* perm_ws,
                                   hipStream_t stream) {
  const int gpr = H / kBlock;
  const int64_t n_groups = (int64_t)T * gpr;
  const int64_t nc = n_chunks_of(T);
  if (nc > 1) {
    const int64_t blocks = nc + (n_groups + kSortThreads / 16 - 1) / (kSortThreads / 16);
    int32_t* counts = static_cast<int32_t*>(perm_ws);
    if (blocks * kSortThreads > 0xffffffffll) {  // too many threads for one grid
      moe_status_t st = moe_quant_act(x, T, H, qx, sx, stream);
      if (st == MOE_OK) st = launch_count(topk_ids, T, k, E, counts, dev_status, stream);
      if (st != MOE_OK) return st;
      return launch_scatter(topk_ids, T, k, E, offsets, sorted_src, dest_row, counts, tiles, stream);
    }
    MOE_LAUNCH("quant_count", quant_count_kernel, dim3((unsigned)blocks), dim3(kSortThreads), 0, stream, topk_ids, T, k,
               E, (int)nc, counts, dev_status, x, n_groups, gpr, qx, sx);
    const moe_status_t st = check_launch("layer prologue");
    if (st != MOE_OK) return st;
    return launch_scatter(topk_ids, T, k, E, offsets, sorted_src, dest_row, counts, tiles, stream);
  }
  const bool tiny = T * k <= kTinySlots;
  const int threads = tiny ? 256 : kSortThreads;
  const int64_t blocks = 1 + (n_groups + threads / 16 - 1) / (threads / 16);
  if (tiny) {
    MOE_LAUNCH("layer_prologue", layer_prologue_kernel<true>, dim3((unsigned)blocks), dim3(threads), 0, stream,
               topk_ids, T, k, E, offsets, sorted_src, dest_row, dev_status, x, n_groups, gpr, qx, sx, tiles);
  } else {
    MOE_LAUNCH("layer_prologue", layer_prologue_kernel<false>, dim3((unsigned)blocks), dim3(threads), 0, stream,
               topk_ids, T, k, E, offsets, sorted_src, dest_row, dev_status, x, n_groups, gpr, qx, sx, tiles);
  }
  return check_launch("layer prologue");
}

}  // namespace moe

using namespace moe;

extern "C" size_t moe_permute_workspace(int32_t T, int32_t k, int32_t E) {
  (void)k;
  if (T < 0 || E <= 0) return 0;
  const int64_t nc = n_chunks_of(T);
  if (nc <= 1) return 256;
  return (size_t)(2 * nc * (E + 1) * sizeof(int32_t) + 256);
}

extern "C" moe_status_t moe_permute(const int32_t* topk_ids, int32_t T, int32_t k, int32_t E,
                                    int32_t* expert_offsets, int32_t* sorted_src, int32_t* dest_row,
                                    int32_t* dev_status, void* ws, size_t ws_bytes, hipStream_t stream) {
  if (T < 0 || E < 1 || E > kMaxExperts || k < 1 || k > kMaxTopk || k > E)
    return fail(MOE_ERR_INVALID_ARG, "moe_permute: T=%d k=%d E=%d (need T>=0, 1<=k<=min(E,32), 1<=E<=1024)", T, k,
                E);
  if ((int64_t)T * k > 0x7fffffff) return fail(MOE_ERR_UNSUPPORTED_SHAPE, "moe_permute: T*k overflows int32");
  if (!expert_offsets || (T > 0 && (!topk_ids || !sorted_src || !dest_row)))
    return fail(MOE_ERR_INVALID_ARG, "moe_permute: null pointer");
  const int64_t nc = n_chunks_of(T);
  if (nc <= 1) {
    if (T * k <= kTinySlots) {
      MOE_LAUNCH("permute_small", permute_small_kernel<true>, dim3(1), dim3(256), 0, stream, topk_ids, T, k, E,
                 expert_offsets, sorted_src, dest_row, dev_status);
    } else {
      MOE_LAUNCH("permute_small", permute_small_kernel<false>, dim3(1), dim3(kSortThreads), 0, stream, topk_ids, T, k,
                 E, expert_offsets, sorted_src, dest_row, dev_status);
    }
    return check_launch("moe_permute");
  }
  const size_t need = moe_permute_workspace(T, k, E);
  if (!ws || ws_bytes < need)
    return fail(MOE_ERR_WORKSPACE, "moe_permute: workspace %zu bytes < %zu", ws_bytes, need);
  if (!aligned(ws, 4)) return fail(MOE_ERR_INVALID_ARG, "moe_permute: misaligned workspace");
  int32_t* counts = static_cast<int32_t*>(ws);
  const moe_status_t st = launch_count(topk_ids, T, k, E, counts, dev_status, stream);
  if (st != MOE_OK) return st;
  return launch_scatter(topk_ids, T, k, E, expert_offsets, sorted_src, dest_row, counts, TilesOut{}, stream);
}
