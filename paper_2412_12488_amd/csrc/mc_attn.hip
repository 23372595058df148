// Paged prefix-prefill attention for gfx950 (CDNA4): attention of the new token
// range [begin, end) of each sequence over the KV already in its pages plus the
// new range itself (paper Sec. 3.1 start_generate, Sec. 3.3 split prefill,
// Sec. 3.4 attention(qkv_data)), and the planning step that precedes it
// (Sec. 3.4 begin_forward: plan the metadata once for all layers).
//
// Work
//   * plan_kernel cuts the ragged batch into work items: a q tile (128 rows = TOK
//     tokens x G query heads of one kv head's group, TOK = 128/G, token-major; 256
//     rows when the KV ranges are long, 32 or 16 when new tokens are few) over a range of 64-key KV tiles - the whole
//     range, or a chunk of it when the batch alone would not fill the GPU (decode
//     steps, short ranges over long contexts), or the prefix that neighbouring
//     sequences with short new ranges share (Sec. 3.4; fork_sequence, Sec. 3.5).
//     Items are ordered longest first; each record holds what the kernel needs to
//     start its first copies.
//   * attn_kernel: one workgroup (4 wavefronts of 64) per (item, kv head), so every
//     K/V byte staged in LDS serves the whole GQA group.  Items that cover a whole
//     range write out/lse; the others write partial rows, which the last of a q
//     tile's items to finish weighs together by their log-sum-exp (where that would
//     take longer than a launch: merge_kernel).  Items of at most 16 rows (decode
//     steps; 32 where new tokens are few) go another way through the kernel,
//     few_rows_item.
// Kernel shape
//   * the KV loop walks 64-key tiles (4 pages) through the page table; each page
//     contributes one contiguous 4 KiB run of K and one of V for this kv head.
//   * S^T = K Q^T on v_mfma_f32_32x32x16 (A = K rows from LDS, B = Q held in
//     registers): a lane then owns ONE query row (column l%32) and 16 keys per
//     32-key chunk, so the softmax row max / row sum are in-lane plus one
//     exchange with lane l^32, and the rescale factor is a per-lane scalar.  With
//     bf16 the row's reference score is fixed after the first half tile (no row max
//     or rescale per tile; a pass whose sums left the safe range is repeated with
//     the moving reference).
//   * O^T += V^T P^T: P^T is the B operand straight from the S^T accumulators
//     (no LDS round trip); V^T comes from LDS with ds_read_b64_tr_b16, which
//     transposes 4 keys x 16 d per 16-lane group on the way in.
//   * LDS tiles are XOR-swizzled so both the row reads (K) and the transposing
//     reads (V) spread over all banks.
#include <math.h>

#include <algorithm>
#include <atomic>
#include <mutex>
#include <type_traits>

#include "mc_common.h"

namespace {

using mc::kHeadPageBytes;
using mc::kPage;
using mc::kRowBytes;

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef int32_t i32x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kBM = 128;       // rows (token x head-in-group) per workgroup
constexpr int kBN = 64;        // keys per KV tile
constexpr int kThreads = 256;  // 4 wavefronts, 32 rows each
constexpr int kPlanThreads = 1024;      // threads of the planner's one workgroup ...
constexpr int kPlanThreadsSmall = 256;  // ... and for batches of few sequences and q tiles
constexpr int kBuckets = 1024;   // of item lengths, for their order (beyond 1023 tiles, 2, 4 ... share one)
constexpr int32_t kPlanMagic = 0x6d63706c;

struct PlanHeader {
  int32_t magic;
  int32_t heads;      // head_counts of the plan
  int32_t num_items;  // work items (q tile x KV chunk) in the work list
  int32_t tile_tokens;
  int32_t batch;
  int32_t total_q;
  int32_t num_merges; // merge records: q tiles whose KV range was cut into several chunks
  int32_t chunk_tiles;  // chunk length the planner settled on (KV tiles); 0 = nothing was cut
  int32_t num_groups_rows;  // partial rows written by shared-prefix items (0 = no groups)
  int32_t tail_chunks;  // chunks per q tile of the remainder round (0 = not applied)
  int32_t arrive_words; // arrival words per merge record and kv head (see MergeRec)
  int32_t err;        // mc_status found on the device by the plan kernel
  int32_t pad[4];
};
static_assert(sizeof(PlanHeader) == 64, "header is 64 bytes");

// Both head counts in one word: where merge records, partial rows and arrivals lie follows from them, so a
// plan made for others is not this batch's, even where its q tiles hold as many tokens (16 are 128 rows of 8
// q heads a kv head, and 16 rows of one).
__host__ __device__ constexpr int32_t head_counts(int32_t hkv, int32_t G) { return (int32_t)((uint32_t)hkv * 16 + G); }

// One work item: q tile (seq, row0) over the KV tiles [t0, t1) of its sequence.  t0 is even.
// chunk < 0: the item covers the tile's whole KV range and writes out/lse itself.  Otherwise it is
// that chunk of the tile `merge` describes: its result (O normalised within the chunk, fp32, and the
// chunk's LSE) is combined with the other chunks' by whichever item comes last (see MergeRec).
// kItemGroup: a shared-prefix item.  Its rows are the ntok new tokens (neighbours in the q array) of
// consecutive sequences whose page tables begin with the same pages as sequence seq's; it covers tiles
// of that common prefix (all of it visible to every row) and is always a chunk.  Its members' merge
// records follow one another from `merge` on.
// The record also carries what the kernel needs to start its first copies without further
// look-ups (each would be one more dependent memory round trip before the first tile): the
// tile's first token in the q array and its token count, where the sequence's page table starts,
// the last table entry the plan has validated for the sequence (as far as the item can reach it:
// which entry of tile t1 - 1 that is), and the page ids of table entries 4 t0 .. 4 t0 + 7
// (clamped to that last entry).
struct ItemRec {
  int32_t seq, row0;
  uint32_t t0_ntok;   // t0 / 2 (24 bits), ntok - 1
  uint32_t t1_flags;  // t1 (26 bits), last validated entry of tile t1 - 1 (2 bits), kItemGroup
  int32_t chunk, q_first, table_off;
  int32_t merge;      // the tile's (of a group: the first member's) merge record
  int32_t ids[8];
};
static_assert(sizeof(ItemRec) == 64, "item record is 64 bytes");
constexpr uint32_t kItemGroup = 1u << 28;

// One q tile of several chunks: nsplit of its own KV range and, if its sequence belongs to a
// shared-prefix group, g_nsplit of the prefix, which the g_stride new tokens of the group's members
// share (g_off: the tile's first among them).  Partial rows are kept per chunk and kv head: the
// R = ntok x G (of the prefix: g_stride x G) rows of chunk c and kv head h start at row
// (part + c ntok) hq + h R (of the prefix: (g_part + c g_stride) hq + h R) of the partial arrays.
//   * Chunks of up to kFlatRows rows (decode steps), of narrow q tiles of up to kNarrowRows: every item
//     writes its rows and counts itself; the last one reads all the others'.
//   * Chunks of more rows: a binary tree over the chunks.  Of two neighbours the first to be done
//     writes its rows and ends, the second reads them, combines, and goes on one level up: of n chunks n - 1
//     are written and read (up to twice as many written, where neighbours miss each other), but not by one
//     workgroup after each other, and the last one up has the tile's result in registers.  These rows
//     are kept as the registers lie, 16 bytes of every row together (by_reg below).
//   * With a group, the prefix's chunks are counted one by one beside the tile's own (a tree's counting
//     as one), and the last of them combines.  Their rows lie row by row.
//   * What the launch would combine too slowly merge_kernel combines, in a launch of its own behind it: the
//     chunks of members of groups and of trees, as the host's rules below say.  These rows lie row by row
//     (a tree's result beside a group's excepted).
// Which chunk comes last differs from run to run; the sums and their order do not.
struct MergeRec {
  int32_t q_row;   // index of the tile's first token among all new tokens of the batch
  int32_t ntok, nsplit, part;
  int32_t g_nsplit, g_part, g_stride, g_off;
};
static_assert(sizeof(MergeRec) == 32, "merge record is 32 bytes");
constexpr int kFlatRows = 16, kNarrowRows = 32;
constexpr int kGroupsBehind = 1, kTreesBehind = 2;   // what is left to merge_kernel
// Whether chunks of shared prefixes are combined inside the attention launch: host, plan and kernel agree
// by the batch's numbers alone.  Few sequences, and no more new tokens than those (some may be idle), which
// share a prefix in items of about kFlatRows rows.  A workgroup reads partial rows at 30 GB/s or so, and the last item
// of a prefix may find every member waiting: items of all rows leave it alone for longer than a launch
// takes.  Append + attention of a layer, 32 / 8 heads, combined in the launch / behind it: 24 forks
// of a 2304-token prompt, 20 us more for the last item / 5 for the launch; 4 forks of 1024 tokens with 4 new ones
// each 30.1 / 18.6 us, with 8 48.8 / 20.1, 8 with 4 45.4 / 20.8; 8 / 1 heads, 8 with 4 49.2 / 19.0.  (Nor do a
// tree over the prefix's chunks, 2.4 to 3.7 us a level, or items of 16 rows in larger batches, which read the
// prefix again, make up for it: 64 forks 48, 50 us a layer instead of 45; 12 forks of 1920 tokens with 53..445
// of their own 30, 20 instead of 20.)
constexpr int kGroupsInLaunch = 8;
__host__ __device__ constexpr bool groups_in_launch(int32_t batch, int32_t total_q) {
  return batch <= kGroupsInLaunch && total_q <= batch;
}
// Whether trees are left to merge_kernel, where groups may bring that launch anyway: if the q tiles x kv heads are so
// few that a tile has many chunks, whose levels follow one another, 2 to 3 us each: up to a 12th of the slots (42).
// Append + attention of a layer, by trees / behind, over 700, 1500, 5000 keys: 40 (4 x 40 tokens) 22.3 / 23.4, 27.1 /
// 25.2, 47.2 / 41.1; 48 (12 x 16) 23.5 / 24.8, 35.7 / 35.4, 65.4 / 64.0; 80 (8 x 40) 24.1 / 27.3, 33.6 / 35.5, 59.0 /
// 60.9.  (Without groups a launch for trees alone costs 3.5 to 4.6 us a layer.  It paid up to a 64th of the slots,
// where narrow q tiles, whose chunks are counted, have taken the trees' place.)
inline bool trees_behind(int64_t tiles, int slots) { return tiles * 12 <= slots; }
// Arrivals: per merge record and kv head arrive_words words that the plan clears.  Word 0 counts
// (and wraps to 0 with the last arrival), the others are the tree, one bit a node (set by the first of
// two, cleared by the second).  They fill the end of the partial LSE array from its last word
// downwards, for which the planner leaves rows of that array (hq >= hkv words each) unused.

constexpr int kCuTilesInLds = 1024;
constexpr int kValidateInPlan = 256;  // batches up to this have their page ids checked by plan_kernel
constexpr int kSpreadItems = 2048;    // items up to which they are written one a thread
constexpr int kTailTilesMax = 2048;   // q tiles up to which the remainder round is looked at
constexpr int kMinSharedTiles = 8;    // a shared prefix shorter than 512 tokens is not worth a group
// Shortest piece a KV range is cut into.  A piece walks its tiles one after the other, a memory
// latency each, and every piece costs a partial row (fp32) for each of its rows, written and read.
// Decode steps (at most one new token a sequence) have few rows: short pieces, 2 tiles as long as
// a row then has no more than the kMergeAhead pieces that a merge requests early, else 4, if
// they pay (short_pieces_pay).  Ranges of more tokens keep 8.  Append + attention of a layer, 32 / 8
// heads, pieces of 8 / 4 / 2 tiles: decode of 1 x 1024 tokens 12.6 / 10.3 / 9.3 us, 1 x 1100 12.6 / 10.3 /
// 10.1, 1 x 2048 12.8 / 10.5 / 10.6, 1 x 4096 13.0 / 11.9 / 13.8, 4 x 1024 13.2 / 11.2 / 10.6, 4 x 2048 15.4 /
// 13.7 / 14.3; ranges of more tokens, 8 or whole / 4 (6 where that would be more items than run at once):
// prefill of 512 17.8 / 17.5, 2 x 512 19.4 / 21.7, 4 x 512 26.2 / 31.3, 1024 25.1 / 26.2, 64 over 448 15.3 / 15.7;
// 256 over 256, 8 / 8 heads, 17.1 / 16.5.
constexpr int kMinChunkTiles = 8, kMinChunkTilesDecode = 4, kMinChunkTilesShort = 2;
constexpr int kNarrowBatch = 16;      // sequences of a batch that may have narrow tiles
// Narrow tiles of ranges up to this are not cut.  16 rows, whole / pieces of 4, us a layer: 32 tokens over 512 15.3 /
// 16.9, over 1024 (17 tiles) 19.7 / 17.9.
constexpr int kWholeNarrow = 12;
constexpr int kMergeAhead = 8;        // partial rows a merge of few rows requests beside their LSEs
// ... and a merge of a shared prefix's rows, for which its pieces are so long that they and the member's own
// one are no more, up to pieces of as many tiles.  Append + attention of a layer, 32 / 8 heads, pieces of 4 / 6 /
// 8 / 12 / 16 tiles: 2 forks of 2048 tokens 12.8 / 13.6 / 14.7 / 16.8 / 19.0 us, of 4096 16.6 / 14.9 / 16.0 / 18.3 /
// 20.7, of 8192 22.9 / 19.2 / 19.8 / 19.1 / 21.8, of 16384 26.7 / 29.2 / 25.6 / 23.1 / 24.9; 8 of 2048 14.5 / 15.2 /
// 15.8 / 17.9 / 20.1, of 4096 19.8 / 17.0 / 17.7 / 19.6 / 21.6, of 8192 29.1 / 23.5 / 22.8 / 21.0 / 22.9.
constexpr int kListedAhead = 12;
constexpr int kRoundsWanted = 4;      // cut only while the launch has fewer items than 4 per slot
// ... and then aim for about one item per slot: measured best on decode batches and on 500-token
// ranges over long contexts (more chunks mean more partial rows to write and merge)
constexpr int kItemsPerSlot = 1;

struct WorkspaceLayout {
  size_t cu_tiles, items, merges, part_lse, part_o, total;
  int32_t max_tiles, max_items, part_cap, batch;
};

inline size_t round64(size_t x) { return (x + 63) & ~size_t(63); }

// The attention kernel comes with q tiles of 128 rows (two workgroups per compute unit) and of
// 256 rows (one, with every K/V fragment read from LDS feeding two MFMAs), the wide ones paying
// off on long KV ranges only.  The planner chooses (it sees the lengths, the host does not) and
// says so in the plan's header; the host only rules the wide tiles out where the batch cannot
// want them - fewer than 4096 new tokens per sequence on average, or fewer wide tiles than four
// per compute unit of a 256-unit GPU - and otherwise launches both kernels, of which the one
// the plan was not made for returns at once.  The workspace is laid out for the tiles of 128 rows
// (more of them), which holds either plan.
inline bool wide_tiles_allowed(int32_t batch, int32_t total_q, int G, int num_kv_heads) {
#ifdef MC_WIDE_TILES
  return MC_WIDE_TILES;
#endif
  const int64_t wide_tiles = ((int64_t)total_q * G + 2 * kBM - 1) / (2 * kBM);
  return batch > 0 && total_q / batch >= 4096 && wide_tiles * num_kv_heads >= 1024;
}
constexpr int kWideMinKeys = 8192;   // mean keys per new token from which the planner goes wide

constexpr int kMaxSlots = 1024;   // 512 compute units: beyond any GPU this library is written for
constexpr size_t kPartialBytesCap = size_t(128) << 20;

// Token rows the partial arrays can hold: the planner cuts KV ranges only as far as this
// allows.  None when the batch has so many q tiles that no GPU would need a cut; otherwise two
// chunks for every new token plus room for the many chunks of a few decode rows, within 128 MiB.
inline int32_t partial_capacity(int32_t total_q, int32_t tile_tokens, int32_t num_q_heads,
                                int32_t num_kv_heads) {
  const int64_t tiles = ((int64_t)total_q + tile_tokens - 1) / tile_tokens;
  if (tiles * num_kv_heads >= (int64_t)kRoundsWanted * kMaxSlots) return 0;
  const int64_t want = 2ll * total_q + 4096;
  const int64_t fit = (int64_t)(kPartialBytesCap / (sizeof(float) * num_q_heads * (mc::kHeadDim + 1)));
  return (int32_t)(want < fit ? want : fit);
}

// part_limit >= 0 caps the rows of the partial arrays below what partial_capacity asks for (a
// caller with a fixed amount of memory): the planner then cuts KV ranges less, or not at all.
inline WorkspaceLayout workspace_layout(int32_t batch, int32_t total_q, int32_t tile_tokens,
                                        int32_t num_q_heads, int32_t num_kv_heads,
                                        int32_t part_limit = -1) {
  WorkspaceLayout w;
  w.max_tiles = (int32_t)(((int64_t)total_q + tile_tokens - 1) / tile_tokens + batch);
  w.part_cap = partial_capacity(total_q, tile_tokens, num_q_heads, num_kv_heads);
  if (part_limit >= 0 && part_limit < w.part_cap) w.part_cap = part_limit;
  w.batch = batch;
  // every extra chunk holds at least one partial row; a shared-prefix group adds items too
  w.max_items = w.max_tiles + w.part_cap + batch;
  w.cu_tiles = sizeof(PlanHeader);
  w.items = w.cu_tiles + round64(sizeof(int32_t) * ((size_t)batch + 1));
  w.merges = w.items + sizeof(ItemRec) * (size_t)w.max_items;
  w.part_lse = w.merges + round64(sizeof(MergeRec) * (size_t)w.max_tiles);
  w.part_o = w.part_lse + round64(sizeof(float) * (size_t)w.part_cap * num_q_heads);
  w.total = w.part_o + sizeof(float) * (size_t)w.part_cap * num_q_heads * mc::kHeadDim;
  return w;
}

// ---------------------------------------------------------------- plan ------
struct PlanArgs {
  const int32_t* cu_q;
  const int32_t* begin;
  const int32_t* page_table;
  const int32_t* cu_pages;
  PlanHeader* hdr;
  int32_t* cu_tiles;
  ItemRec* items;
  MergeRec* merges;
  int32_t batch, total_q, tile_tokens, num_pages, max_tiles, max_items, max_merges, part_cap;
  uint32_t* arrivals_end;  // one past the last arrival word (see MergeRec)
  int32_t hq, hkv, slots;   // q and kv heads; workgroups the GPU runs at a time
  int32_t allow_groups; // look for decode rows of neighbouring sequences that share a prefix
  int32_t ahead;        // tokens every sequence's begin may still grow by while the plan is in use
  int32_t wide_tile_tokens, slots_wide;   // the wide q tiles, if the host allows them (else 0)
};

// Scans over a wavefront by data-parallel moves (rows of 16 lanes, then the rows' last lanes): no LDS
// permutes, of which a scan of shuffles is six in a row.  The planner is one workgroup whose steps
// follow one another, so their latency is its time.  With the wider page-id loads, the tile kept by its
// thread and 1024 buckets instead of 4096, the plan of one decode row takes 11.5 -> 10.3 us, of 256 new
// tokens over 256 8.4 -> 7.2, of 256 decode rows 20.9 -> 20.1 (under the profiler).
template <typename Op>
__device__ __forceinline__ int wave_inclusive(int x, int identity, Op&& op) {
  x = op(x, __builtin_amdgcn_update_dpp(identity, x, 0x111, 0xf, 0xf, false));   // row_shr:1
  x = op(x, __builtin_amdgcn_update_dpp(identity, x, 0x112, 0xf, 0xf, false));
  x = op(x, __builtin_amdgcn_update_dpp(identity, x, 0x114, 0xf, 0xf, false));
  x = op(x, __builtin_amdgcn_update_dpp(identity, x, 0x118, 0xf, 0xf, false));
  x = op(x, __builtin_amdgcn_update_dpp(identity, x, 0x142, 0xa, 0xf, false));   // row_bcast:15
  x = op(x, __builtin_amdgcn_update_dpp(identity, x, 0x143, 0xc, 0xf, false));   // row_bcast:31
  return x;
}
__device__ __forceinline__ int wave_inclusive_sum(int x) {
  return wave_inclusive(x, 0, [](int p, int q) { return p + q; });
}
__device__ __forceinline__ int wave_inclusive_max(int x) {
  return wave_inclusive(x, INT32_MIN, [](int p, int q) { return max(p, q); });
}

// Block-wide exclusive scan of N values per thread at once (NT threads): the wavefront totals through
// LDS (N x NT / 64 ints), two barriers in all.
template <int NT, int N>
__device__ __forceinline__ void block_exclusive_scan_n(int (&v)[N], int* lds, int (&total)[N]) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  int incl[N];
#pragma unroll
  for (int k = 0; k < N; ++k) incl[k] = wave_inclusive_sum(v[k]);
  __syncthreads();               // earlier readers of lds are done
  if (lane == 63)
#pragma unroll
    for (int k = 0; k < N; ++k) lds[k * (NT / 64) + wave] = incl[k];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < N; ++k) {
    int before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) {
      const int x = lds[k * (NT / 64) + w];
      if (w < wave) before += x;
      all += x;
    }
    total[k] = all;
    v[k] = before + incl[k] - v[k];
  }
}
template <int NT>
__device__ __forceinline__ int block_exclusive_scan(int v, int* lds, int* total) {
  int one[1] = {v}, sum[1];
  block_exclusive_scan_n<NT>(one, lds, sum);
  *total = sum[0];
  return one[0];
}

// Block-wide sum of one value (0 .. 2^63 - 1) per thread, to every thread: in three pieces of 21 bits
// (lds holds 3 x NT / 64 ints).
template <int NT>
__device__ __forceinline__ long long block_sum(long long v, int* lds) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  int piece[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) piece[k] = wave_inclusive_sum((int)(v >> (21 * k)) & 0x1fffff);
  __syncthreads();               // earlier readers of lds are done
  if (lane == 63)
#pragma unroll
    for (int k = 0; k < 3; ++k) lds[3 * wave + k] = piece[k];
  __syncthreads();
  long long all = 0;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w)
    all += lds[3 * w] + ((long long)lds[3 * w + 1] << 21) + ((long long)lds[3 * w + 2] << 42);
  return all;
}

// The same of values whose sum is below 2^31.
template <int NT>
__device__ __forceinline__ int block_sum_int(int v, int* lds) {
  const int t = threadIdx.x, sum = wave_inclusive_sum(v);
  __syncthreads();               // earlier readers of lds are done
  if ((t & 63) == 63) lds[t >> 6] = sum;
  __syncthreads();
  int all = 0;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) all += lds[w];
  return all;
}

// Block-wide inclusive running maximum of one value per thread.
template <int NT>
__device__ __forceinline__ int block_inclusive_max_scan(int v, int* lds) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int incl = wave_inclusive_max(v);
  __syncthreads();
  if (lane == 63) lds[wave] = incl;
  __syncthreads();
  int before = INT32_MIN;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w)
    if (w < wave) before = max(before, lds[w]);
  return max(before, incl);
}

// Whether pieces of L < kMinChunkTiles tiles gain more than they cost over pieces of kMinChunkTiles
// (over whole ranges, if the longest has no more).  us of append + attention of a layer with pieces of
// 8 (whole) / of L tiles; heads q / kv:
//   - All items have to run at once: the ones left over take a turn of their own.  616 items for 512
//     slots, 32 x 64..900 tokens, 32 / 8, L = 4: 23.1 / 23.4.  (The count is an estimate, up to a tenth
//     above the true one.)  An eighth more than the slots is made up for if the pieces are not the
//     shortest nor many a row, and no group's merges grow: 560 items, 24 x 300..1000, 32 / 8, which the
//     estimate puts beyond that, L = 4: 24.2 / 24.0; 672 items, 48 forks of a 512-token prompt with 48..888
//     of their own, 32 / 8, L = 6: 31.6 / 30.7.
//   - Rows of more than 24 pieces: half the slots.  8 / 2 heads, 8192 tokens, L = 4: 1 row 13.6 / 12.8, 4
//     rows (256 items) 16.1 / 16.7, 8 rows (512) 21.0 / 22.2; 6000 tokens (24 pieces), 8 rows (384) 18.5 / 19.6.
//   - A merge reads every partial row: 8 heads, one of them kv, forks of a 4096-token prompt, L = 4: 64 rows
//     21.5 / 20.4, 128 23.5 / 23.4.
//   - Pieces of 6 differ from those of 8 in how well they fill the slots only, and add rows to a group's
//     merges: 32 / 8 heads, 8 x 1024..4096 tokens (392 items) 23.3 / 23.1, 6 (328) 19.3 / 22.3; 8 / 2,
//     128 forks of 2048 tokens 22.6 / 21.3, L = 4 20.8.
//   - Whole ranges have nothing to combine: what is saved, longest - L tiles of latency, has to outweigh
//     that, and the items that then read at once.  32 / 8 heads: 24 x 64..500 tokens, L = 4, 15.5 / 16.0, L = 2:
//     16 x 320 12.5 / 13.4, 20 x 320 13.1 / 14.5, 16 x 200 11.4 / 12.5; 8 / 2: 64 x 64..500 13.7 / 13.9; 8 / 1:
//     128 x 100..512 13.9 / 14.5, 160 x 100..300 12.5 / 13.8.
// The lines were drawn where one wavefront walked an item's tiles and a launch combined the chunks, which
// made whole ranges of up to 8 tiles up to 2 us slower than they are now; so short pieces are still
// taken where they now lose a little (24 x 64..500, 16 x 320, 64 x 64..500, 128 x 100..512; 4 x 8192, 8 x 6000).
// cost: tiles of all the ranges, at most 8 x slots / hkv.  No division: this is part of every step's
// plan.  A q tile has kBM rows, so q heads are kv heads x kBM / tile_tokens.
__device__ __forceinline__ bool short_pieces_pay(const PlanArgs& a, int L, int longest, bool groups, int tiles,
                                                 int cost) {
  // items x 2 L; a range's last piece has half of L on average
  const int items = (2 * cost + tiles * L) * a.hkv, full = 2 * L * a.slots;
  const bool many = longest > 24 * L;
  const int share = groups || many || L < kMinChunkTilesDecode ? 17 : 18;      // of 16
  if (16 * items > share * (many ? full / 2 : full)) return false;
  const int whole = tiles * a.hkv;                               // of q heads: whole x kBM / tile_tokens
  if ((float)whole * (float)longest > 96.f * (float)(L * a.tile_tokens)) return false;     // 12288 / kBM
  if (L > kMinChunkTilesDecode && (groups || 8 * items < 7 * full)) return false;
  const int saved = longest - L;
  return longest > kMinChunkTiles || whole <= min(8 + 64 * (saved - 1), (1 + 2 * saved) * a.tile_tokens);
}

// The header of a plan that the attention has nothing to do for.
__device__ __forceinline__ void refuse_plan(PlanHeader* h) {
  h->err = MC_ERR_RANGE;
  h->num_items = h->num_merges = 0;
  h->magic = kPlanMagic;
}

// The rows of a q tile of a batch of few sequences and few new tokens: kBM, or kNarrowRows or half as many, whose
// items few_rows_item walks with all four wavefronts, cut into pieces of `pieces` KV tiles.  tiles: the batch's tiles of
// kBM rows, of kNarrowRows, of half as many; visits: the KV tiles they look at, as if all of a sequence's tiles lay
// in its middle; longest: KV tiles of the longest range; many: of the longest of more than kFlatRows rows (0: none).
// A workgroup alone on its compute unit takes 0.74 us for a KV tile and 128 rows, 0.56 us for 32 and 0.60 for 16 (each
// wavefront walks every fourth half tile).  So narrow tiles have a third of the rate, but need no tree of
// chunks (2 to 3 us a level) and no launch behind, and fill the compute units where q tiles of 128 rows are few.  On
// all units that is 15 TB/s, what the L2s hand out, and two workgroups a unit take 1.08 and 1.04 us: there are never
// more narrow items than compute units.
// Narrow tiles are taken as follows (us a layer of four: append, attention, their share of the plan; 32 / 8 heads
// unless named; tokens over keys cached).
//   - 16 rows up to 18 KV tiles, uncut, or up to 16 a compute unit if every tile can be cut at least once.  Whole
//     tiles / 32 rows / 16 rows: 64 over 512 19.1 / 17.9 / 13.9; 128 over 1024 23.9 / 20.2 / 19.4; 8 over 4096 22.0 /
//     25.0 / 17.7, over 16000 30.4 / 33.4 / 24.9; 32 over 1024 21.5 / 18.2 / 15.4, over 4096 25.0 / 21.7 / 22.8, over
//     8192 28.2 / 26.3 / 33; 64 over 2048 27.0 / 22.0 / 23.0.
//   - 32 rows up to 24 KV tiles a compute unit.  64 over 4096 31.0 / 26.2; 128 over 4096 (32 tiles) 33.6 / 35.1.
//   - Both only if whole tiles would not be done sooner.  Estimates, in the time of a narrow item's KV tile, with the
//     weights that part the figures below (and more like them, 64 / 8 to 8 / 1 heads, 5 to 1000 tokens): narrow ones
//     take the longest piece, and 9 (32 rows) or 5 more if pieces have to be combined.  Whole ones are cut into pieces
//     of 8 KV tiles or more, two for a KV tile of many rows and 5 for a level of their tree (2 with up to 64 rows); one
//     for a KV tile of few rows, and 5 to combine those.  That counts where lengths differ: narrow pieces have one
//     length for all ranges, and one workgroup a compute unit leaves few of them.  Whole / narrow: 15 rows over
//     500..4096 beside 800 tokens, 8 / 2 heads, 26.0 / 44.9; 8 rows over 4000 beside 100 tokens over 900 45.0 / 61.7; 4
//     rows over 300..1100 beside 200 tokens 18.7 / 20.1, over 600..1500 beside 100 18.9 / 17.3.  One range: 128 over
//     2300 28.6 / 27.3, over 2700 29.2 / 29.6; 256 over 1100 24.5 / 23.5, over 1250 24.8 / 24.7; 64 over 3000, 64 / 8
//     heads, 28.5 / 29.8.
//   - Always up to a 64th of the slots of (q tile, kv head) pairs if the longest range has many rows: whole tiles have
//     many chunks there, and their trees take longer.  Whole with trees / with a launch behind / narrow: 32 over 8192
//     35.5 / 28.3 / 26.4, over 16000 45.9 / 34.7 / 35.9; 128 over 32000, 8 / 1 heads, 55.4 / 43.3 / 51.3.  (The launch
//     behind costs 3.5 where ranges are shorter, and the host does not see how long they are.)
// Pieces: as many equal ones a tile as there are compute units for, or by the sum of the lengths, no more than the
// launch's grid has room for.  A tile's last item combines them, 0.5 us for each of 32 rows and half of that for 16,
// eight at a time (nine take as long as 16): so 16 at most, or 8 where those are no more than 4 KV tiles longer (20
// over 9000: 9 of 16 tiles 28.6, 8 of 18 26.4); of 16 rows 32 in long ranges of few tiles (8 over 32000, 8 / 1 heads,
// 31.8 -> 27.5; with more tiles, 16 over 32000, 32.9 -> 35.8).
// Every line of the planner runs once, from memory, and its length is its time: both sizes are weighed at once, 16 rows
// in odd lanes and 32 in even ones, in floats, and neither the lengths' exact sum nor paths that such a batch cannot
// take are in its planner.  (A form in integers, once a size, made a plan 2.4 us longer than the two rules by sums
// alone did; this makes it 1 us shorter.)
__device__ __forceinline__ int narrow_rows(const PlanArgs& a, const int* tiles, const int* visits, int longest, int many,
                                           int& pieces) {
  const bool half = threadIdx.x & 1;             // 16 rows in odd lanes, 32 in even ones
  const int n0 = tiles[0], n = tiles[1 + half], units = a.slots / 2, items = n * a.hkv;
  const float all = (float)visits[1 + half] * a.hkv, range = longest;
  auto over = [](float x, float y) { return x * __builtin_amdgcn_rcpf(y); };
  const bool few_pairs = 64 * n0 * a.hkv <= a.slots;
  const bool fits = tiles[2] > n0 && items <= units && n <= min(a.max_items, a.max_merges) && longest <= 1 << 20 &&
                    (half ? longest <= 18 || (2 * items <= units && all <= 16 * units) : all <= 24 * units || few_pairs);
  float L = over(range, floorf(over(units + 0.5f, items)));
  L = fminf(L, over(all, units - items));
  L = fmaxf(L, over(range, half && longest > 256 && 64 * items <= units ? 32 : 16));
  const float eight = ceilf(range * 0.125f);
  L = eight - L > 4 ? L : fmaxf(L, eight);
  const int most = visits[1 + half] + n * (a.total_q / (2 * kBN) + 1);      // KV tiles, from below the diagonal
  L = ceilf(fmaxf(fmaxf(L, kMinChunkTilesDecode), over(most, a.max_items - n) * 1.001f));
  const bool cut = L < range && longest > kWholeNarrow;
  const float narrow = cut ? L + (!half && many > L ? 9 : 5) : range;
  const float per = fmaxf(kMinChunkTiles, over((float)visits[0] * a.hkv, a.slots));
  float whole = fminf(2 * many, 2 * per);
  if (many > per)
    whole += (a.total_q * kBM <= 64 * n0 * a.tile_tokens ? 2 : 5) * ceilf(__log2f(over(many, per)) - 0.01f);
  if (longest > many) whole = fmaxf(whole, fminf(range, per + 5));
  const unsigned long long pays = __ballot(fits && ((few_pairs && longest == many) || narrow <= whole));
  if ((pays & 3) == 0) return kBM;
  const int lane = (pays & 2) != 0;
  pieces = __builtin_amdgcn_readlane((int)fminf(L, range), lane);
  return kNarrowRows >> lane;
}

// Page ids of every needed table entry, for batches too large for the planner's one workgroup
// to walk: one wavefront per sequence, many workgroups.  Runs after plan_kernel and, on a bad
// id, turns its verdict into MC_ERR_RANGE with an empty work list.  (Sequences whose offsets
// are malformed were rejected by the planner already; they are skipped here.)
__global__ __launch_bounds__(256) void validate_pages_kernel(PlanArgs a) {
  const int s = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (s >= a.batch || a.hdr->err != MC_OK) return;
  const int q = a.cu_q[s + 1] - a.cu_q[s], b = a.begin[s];
  const int p0 = a.cu_pages[s], np = a.cu_pages[s + 1] - p0;
  if (q <= 0 || b < 0 || p0 < 0) return;
  const int64_t need64 = ((int64_t)b + q + a.ahead + kPage - 1) / kPage;
  if (need64 > np) return;
  const int need = (int)need64;
  int err = 0;
  for (int i = lane; i < need; i += 64 * 8) {   // eight independent loads per lane and trip
    int32_t pg[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) pg[u] = i + 64 * u < need ? a.page_table[p0 + i + 64 * u] : 0;
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (pg[u] < 0 || pg[u] >= a.num_pages) err = 1;
  }
  if (__ballot(err) != 0 && lane == 0) {
    refuse_plan(a.hdr);
  }
}

// One workgroup.  Validates the ragged-batch arrays, cuts every sequence's new range into q
// tiles of tile_tokens tokens, cuts long KV ranges into chunks when the launch would otherwise
// have too few work items to fill the GPU (decode rows, short batches over long contexts),
// and orders the items by decreasing number of KV tiles (longest first), so that the tail of
// the launch is made of short items.
// NT threads: 1024, or 256 for small batches, whose many block-wide steps then cost a quarter
// of the wavefronts to synchronise.
template <int NT, bool kMayNarrow>
__global__ __launch_bounds__(NT) void plan_kernel(PlanArgs a) {
  __shared__ int scan[5 * NT / 64];   // wavefront totals of the block scans and sums
  __shared__ int hist[kBuckets];
  __shared__ int s_err, s_maxcost, s_table_end, s_pages, s_suspect, s_sums[6], s_many, s_alike;
  // per-sequence arrays of batches that fit: the searches and tile look-ups below stay in LDS
  __shared__ int s_cu[kCuTilesInLds + 1], s_cuq[kCuTilesInLds + 1], s_beg[kCuTilesInLds],
      s_cup[kCuTilesInLds + 1];
  // shared-prefix groups, per sequence: pages in common with the next sequence; prefix tiles the
  // group covers (0 = not in a group); the group's first sequence (-1 = none); at that first
  // sequence the group's new tokens, the base of its partial rows and its last sequence
  __shared__ int s_common[kCuTilesInLds], s_gp[kCuTilesInLds], s_glead[kCuTilesInLds],
      s_gsize[kCuTilesInLds], s_gbase[kCuTilesInLds], s_glast[kCuTilesInLds];
  __shared__ int s_groups;
  // of items written one a thread: tile and place in the list; of a tile: its first item and its merge record
  __shared__ uint16_t s_owner[kSpreadItems], s_place[kSpreadItems];
  __shared__ int s_first[NT], s_merge[NT];
  // remainder round: flags of the q tiles that are cut, the cost bucket at the boundary and how
  // many tiles of it are taken
  __shared__ uint8_t s_tailflag[kTailTilesMax];
  __shared__ int s_tail_bucket, s_tail_take, s_tail_taken;
  const int t = threadIdx.x;
  if (t == 0) { s_err = 0; s_maxcost = 1; s_table_end = s_pages = s_suspect = s_alike = 0; }
  for (int i = t; i < kBuckets; i += NT) hist[i] = 0;
  const bool cu_in_lds = a.batch <= kCuTilesInLds;
  if (cu_in_lds) {
    for (int i = t; i <= a.batch; i += NT) {
      s_cuq[i] = a.cu_q[i];
      s_cup[i] = a.cu_pages[i];
      if (i < a.batch) s_beg[i] = a.begin[i];
    }
  }
  __syncthreads();

  // the batch's offset arrays: from LDS when they fit there (one read of global memory in all)
  auto cuq = [&](int i) { return cu_in_lds ? s_cuq[i] : a.cu_q[i]; };
  auto cup = [&](int i) { return cu_in_lds ? s_cup[i] : a.cu_pages[i]; };
  auto beg = [&](int i) { return cu_in_lds ? s_beg[i] : a.begin[i]; };
  const int per = (a.batch + NT - 1) / NT;
  const int s_lo = min(t * per, a.batch), s_hi = min(s_lo + per, a.batch);
  // 0. q tile width: wide tiles when a new token sees kWideMinKeys keys on average.  Their ranges are not
  //    cut: the host allows them where there are four a compute unit of a 256-unit GPU.
  bool wide = false;
  if (!kMayNarrow && a.wide_tile_tokens > 0) {
    long long keys = 0, rows = 0;
    for (int s = s_lo; s < s_hi; ++s) {
      const long long q = cuq(s + 1) - cuq(s), b = beg(s);
      if (q > 0 && b >= 0) { rows += q; keys += q * b + q * (q + 1) / 2; }
    }
    keys = block_sum<NT>(keys, scan);
    rows = block_sum<NT>(rows, scan);
    if (rows > 0 && keys / rows >= kWideMinKeys) {
      a.tile_tokens = a.wide_tile_tokens;
      a.slots = a.slots_wide;
      wide = true;
    }
  }
  // 1. validate, count tiles per sequence (contiguous chunk of sequences per thread)
  int my_tiles = 0, err = 0, maxcost = 1, my_pages = 0, table_end = 0;
  // (kMayNarrow) the same in tiles of kNarrowRows rows and of half as many, the KV tiles that all three have to look
  // at, and the longest range of more than kFlatRows rows
  const int narrow_tokens = a.tile_tokens * kNarrowRows / kBM;
  int narrow_tiles[2] = {0, 0}, visits[3] = {0, 0, 0}, many = 0;
  if (t == 0 && (cuq(0) != 0 || cuq(a.batch) != a.total_q || cup(0) < 0)) err = 1;
  for (int s = s_lo; s < s_hi; ++s) {
    const int q = cuq(s + 1) - cuq(s), b = beg(s);
    const int np = cup(s + 1) - cup(s);
    if (q < 0 || b < 0 || np < 0 || cuq(s) < 0 || cuq(s + 1) > a.total_q) { err = 1; continue; }
    if (q == 0) continue;
    const int64_t end = (int64_t)b + q + a.ahead;
    if ((end + kPage - 1) / kPage > np) { err = 1; continue; }
    const int need = (int)((end + kPage - 1) / kPage);
    my_pages += need;            // (of all sequences no more than cu_pages[batch])
    table_end = max(table_end, cup(s) + need);
    my_tiles += (q + a.tile_tokens - 1) / a.tile_tokens;
    if constexpr (kMayNarrow) {
      // (q tiles have 2^i tokens, and no more than 2^10 have few enough rows, over 2^20 KV tiles: narrow_rows)
      const int mean = (int)min((end - q / 2 + kBN - 1) / kBN, (int64_t)1 << 20), shift = __builtin_ctz(a.tile_tokens);
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        narrow_tiles[k] = (q + (narrow_tokens >> k) - 1) >> (shift - 2 - k);
        visits[1 + k] = narrow_tiles[k] * mean;
      }
      visits[0] = ((q + a.tile_tokens - 1) >> shift) * mean;
    }
    const int T = (int)((end + kBN - 1) / kBN);
    if (q > narrow_tokens / 2) many = max(many, T);
    maxcost = max(maxcost, T);
  }
  // In the small variant all sequences are the first wavefront's, a thread each: it sums the tiles before them here,
  // ahead of the barrier that there is.
  constexpr bool kFirstWave = NT == kPlanThreadsSmall;
  constexpr int kSums = kMayNarrow ? 6 : 1;
  int before[kSums] = {my_tiles};
  if constexpr (kMayNarrow) {
    for (int k = 0; k < 2; ++k) before[1 + k] = narrow_tiles[k];
    for (int k = 0; k < 3; ++k) before[3 + k] = visits[k];
  }
  if (kFirstWave && t < 64) {
#pragma unroll
    for (int k = 0; k < kSums; ++k) {
      const int incl = wave_inclusive_sum(before[k]);
      before[k] = incl - before[k];
      if (t == 63) s_sums[k] = incl;
    }
    if constexpr (kMayNarrow) {
      many = wave_inclusive_max(many);
      if (t == 63) s_many = many;
    }
  }
  // (one LDS atomic per wavefront, not per thread: 1024 atomics on one address take microseconds)
  if (__ballot(err != 0) != 0 && (t & 63) == 0) atomicOr(&s_err, 1);
  maxcost = wave_inclusive_max(maxcost);
  table_end = wave_inclusive_max(table_end);
  my_pages = wave_inclusive_sum(my_pages);
  if ((t & 63) == 63) {
    atomicMax(&s_maxcost, maxcost);
    atomicMax(&s_table_end, table_end);
    atomicAdd(&s_pages, my_pages);
  }
  __syncthreads();
  if (s_err) {
    if (t == 0) refuse_plan(a.hdr);
    return;
  }
  // 2. page ids of every needed table entry.  Small batches (their offsets sit in LDS) look at the table as it lies
  //    first, from the first sequence's entries to the last needed one, four entries a lane; the first kFlatLoads
  //    loads of a lane are under way until the items are counted (5b).  Only where that finds an id out of range,
  //    which may be one that no token needs, or where more than half of it is not needed, are the sequences' own
  //    entries looked at.  256 decode rows over 1024..4096 tokens: 8.6 us sequence by sequence, now 3.
  typedef int32_t i32x4u __attribute__((ext_vector_type(4), aligned(4)));
  auto bad_id = [&](i32x4u x) {
    const int lo = min(min(x[0], x[1]), min(x[2], x[3])), hi = max(max(x[0], x[1]), max(x[2], x[3]));
    return lo < 0 || hi >= a.num_pages;
  };
  constexpr int kFlatLoads = NT > 256 ? 1 : 4, kFlatTrip = 4;
  const bool ids_here = a.batch <= kValidateInPlan;
  const int table0 = cup(0), table_n = ids_here ? s_table_end - table0 : 0;
  bool suspect = ids_here && (table_n < 4 || table_n / 2 > s_pages);
  i32x4u flat_ids[kFlatLoads];
  // (entries 4 i .. 4 i + 3, or the last four)
  auto flat_load = [&](int i) {
    return *reinterpret_cast<const i32x4u*>(a.page_table + table0 + min(4ll * i, table_n - 4ll));
  };
#pragma unroll
  for (int k = 0; k < kFlatLoads; ++k)
    flat_ids[k] = ids_here && !suspect ? flat_load(t + k * NT) : i32x4u{0, 0, 0, 0};
  auto look_at_rest = [&]() {
    for (int i = t + kFlatLoads * NT; ids_here && !suspect && 4ll * i < table_n; i += kFlatTrip * NT) {
      i32x4u more[kFlatTrip];
#pragma unroll
      for (int k = 0; k < kFlatTrip; ++k) more[k] = flat_load(i + k * NT);
#pragma unroll
      for (int k = 0; k < kFlatTrip; ++k) suspect |= bad_id(more[k]);
    }
  };
  bool looked = false;
  // (batches beyond that: validate_pages_kernel, launched after this kernel, on many workgroups)
  // 3b. shared-prefix groups (Sec. 3.4, fork_sequence in Sec. 3.5: sequences may share the pages of a common
  //     prefix).  The new tokens of neighbouring sequences with short new ranges (decode rows,
  //     or a few tokens each) whose tables start with the same pages attend that prefix together
  //     as one q tile - their tokens are neighbours in the q array, and every key of the prefix
  //     lies before every one of them, so no mask is involved - one K/V read for all of them,
  //     and their own remainders one by one; the parts are merged by LSE like any other chunks.
  //     Prefix items hold the whole group's rows, or where they are combined in the launch (see MergeRec)
  //     those of the members whose first tokens lie in the same kFlatRows rows of it: a slice.
  const bool sliced = !kMayNarrow && groups_in_launch(a.batch, a.total_q);
  const int slice = max(kFlatRows * a.tile_tokens / kBM, 1);
  const bool try_groups = a.allow_groups && cu_in_lds && a.batch >= 2 && a.batch <= NT;
  constexpr int kMinPages = kMinSharedTiles * kBN / kPage;
  // a sequence can be a member if its new range leaves room for another token in a q tile
  auto is_short = [&](int sq) {
    const int q = s_cuq[sq + 1] - s_cuq[sq];
    return q >= 1 && q < a.tile_tokens;
  };
  if (t == 0) s_groups = 0;
  if (try_groups) {
    for (int i = t; i < a.batch; i += NT) { s_common[i] = 0; s_gp[i] = 0; s_glead[i] = -1; s_gsize[i] = 0; }
    __syncthreads();
    // pages in common between s and s+1, among the whole pages cached by both.  First every
    // pair at once, one thread each: unrelated sequences differ in their first page and are
    // done (s_common = 1 marks a pair that is not).  Then 16 lanes a remaining pair, behind the look at the rest of
    // the table, which asks for all of it at once, where a pair's lanes walk it, a memory latency for every 128 entries
    // (plan of 99 forks of 4000 tokens 34.2 us when every sequence's ids were looked at ahead, 38 when all of them were
    // behind, now 30.6; of 64 of 2048 26.9, 24.0, 22.6).
    if (t + 1 < a.batch && is_short(t) && is_short(t + 1) &&
        min(s_beg[t], s_beg[t + 1]) / kPage >= kMinPages &&
        a.page_table[s_cup[t]] == a.page_table[s_cup[t + 1]])
      s_common[t] = s_alike = 1;
    __syncthreads();
    looked = s_alike != 0;
  }
  if (looked) {
    look_at_rest();
    // (16 lanes a pair, eight entries a lane and table in flight: the pairs of 64 sequences in one turn)
    for (int sq = t >> 4; sq + 1 < a.batch; sq += NT >> 4) {
      if (s_common[sq] == 0) continue;
      const int lim = min(s_beg[sq], s_beg[sq + 1]) / kPage;
      const int pa = s_cup[sq], pb = s_cup[sq + 1];
      int common = lim;
      for (int i0 = t & 15; i0 - (t & 15) < common; i0 += 128) {
        int x[8], y[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          x[u] = i0 + 16 * u < lim ? a.page_table[pa + i0 + 16 * u] : 0;
          y[u] = i0 + 16 * u < lim ? a.page_table[pb + i0 + 16 * u] : 0;
        }
        int first = lim;               // the first entry that differs
#pragma unroll
        for (int u = 7; u >= 0; --u)
          if (x[u] != y[u]) first = i0 + 16 * u;
#pragma unroll
        for (int off = 8; off > 0; off >>= 1) first = min(first, __shfl_xor(first, off));
        common = min(common, first);
      }
      if ((t & 15) == 0) s_common[sq] = common;
    }
    __syncthreads();
    // Runs of such sequences linked by enough common pages, cut greedily into groups of at most
    // tile_tokens new tokens.  The thread of a run's first sequence walks the run group by
    // group (cu_q is the prefix sum of the new tokens: the end of a group is a binary search);
    // everything per member is done by the member's own thread.
    const bool mine = t < a.batch;
    auto linked = [&](int sq) {   // sq and sq+1 sit in one run
      return sq >= 0 && sq + 1 < a.batch && is_short(sq) && is_short(sq + 1) &&
             s_common[sq] >= kMinPages;
    };
    const bool in_run = mine && is_short(t) && (linked(t) || linked(t - 1));
    // (unrelated sequences, the usual case: nothing is linked and the rest is skipped)
    if (__ballot(in_run) != 0 && (t & 63) == 0) s_groups = -1;
    __syncthreads();
    const bool any_run = s_groups != 0;
    __syncthreads();
    if (t == 0) s_groups = 0;
    if (any_run) {
      // last sequence of the run a sequence sits in: the nearest j >= t that is not linked to j + 1
      // (a running maximum over the reversed index)
      {
        const int j = a.batch - 1 - t;     // this thread's element of the reversed scan
        const bool ends = j >= 0 && !linked(j);
        const int v = block_inclusive_max_scan<NT>(ends ? -j : INT32_MIN, scan);
        if (j >= 0) s_gbase[j] = -v;       // scratch until step 5: run end of sequence j
      }
      __syncthreads();
      if (in_run && !linked(t - 1)) {      // first sequence of a run
        const int run_end = s_gbase[t];
        for (int lead = t; lead <= run_end;) {
          // the last member: the largest e <= run_end with cu_q[e + 1] - cu_q[lead] <= tile_tokens
          int lo = lead, hi = run_end;
          const int limit = s_cuq[lead] + a.tile_tokens;
          while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (s_cuq[mid + 1] <= limit) lo = mid; else hi = mid - 1;
          }
          if (lo > lead) {                 // two members or more: a group
            s_gsize[lead] = s_cuq[lo + 1] - s_cuq[lead];   // rows of the group's q tile
            s_glast[lead] = lo;
            s_gbase[lead] = INT32_MAX;     // becomes the fewest pages two neighbouring members share
            s_groups = 1;
          }
          lead = lo + 1;
        }
      }
      __syncthreads();
      // every sequence finds the nearest group lead at or before it and checks that it is a member
      const int near = block_inclusive_max_scan<NT>(mine && s_gsize[t] > 0 ? t : -1, scan);
      const bool member = in_run && near >= 0 && t <= s_glast[near];
      if (member && t < s_glast[near]) atomicMin(&s_gbase[near], s_common[t]);
      __syncthreads();
      if (member && t == near)
        s_gbase[t] = (s_gbase[t] / (2 * kBN / kPage)) * 2;   // prefix tiles, even (scratch until step 5)
      __syncthreads();
      if (mine) {
        s_glead[t] = member ? near : -1;
        s_gp[t] = member ? s_gbase[near] : 0;
        if (sliced) {      // from here on in s_common: the tokens of the slice this sequence leads, else 0
          const int first = member ? s_cuq[near] : 0, id = (s_cuq[t] - first) / slice;
          int end = t;
          if (member && (t == near || (s_cuq[t - 1] - first) / slice != id))
            do ++end; while (end <= s_glast[near] && (s_cuq[end] - first) / slice == id);
          s_common[t] = s_cuq[end] - s_cuq[t];
        }
      }
    }
    __syncthreads();
  }
  bool groups = try_groups && s_groups != 0;

  // 3. exclusive scan of tiles per sequence
  //     Tiles of fewer rows where even these are no more than a workgroup a compute unit: narrow_rows.
  int total_tiles, base;
  bool narrow = false;
  int pieces = 0;
  if constexpr (kMayNarrow) {
    const int rows = groups ? kBM : narrow_rows(a, s_sums, s_sums + 3, s_maxcost, s_many, pieces);
    const int k = rows == kBM ? 0 : rows == kNarrowRows ? 1 : 2;
    base = k == 0 ? before[0] : k == 1 ? before[1] : before[2];
    total_tiles = s_sums[k];
    narrow = k > 0;
    if (narrow) a.tile_tokens = narrow_tokens >> (k - 1);
  } else {
    if constexpr (kFirstWave) { base = before[0]; total_tiles = s_sums[0]; }
    else base = block_exclusive_scan<NT>(my_tiles, scan, &total_tiles);
  }
  for (int s = s_lo; s < s_hi; ++s) {
    a.cu_tiles[s] = base;
    if (cu_in_lds) s_cu[s] = base;
    const int q = cuq(s + 1) - cuq(s);
    base += (q + a.tile_tokens - 1) / a.tile_tokens;
  }
  if (t == 0) {
    a.cu_tiles[a.batch] = total_tiles;
    if (cu_in_lds) s_cu[a.batch] = total_tiles;
  }
  __threadfence_block();
  __syncthreads();
  if (total_tiles > (narrow ? a.max_items : a.max_tiles)) {
    if (t == 0) refuse_plan(a.hdr);
    return;
  }

  // q tile i: its sequence, first row, token count, KV tiles, the last even tile index at which
  // a chunk may start (every row must see at least the first key of every chunk), the prefix
  // tiles its shared-prefix group covers, the group's new tokens if this tile leads one, and those of
  // the prefix items that the tile leads
  struct Tile { int s, row0, ntok, T, dmax, pt, gm, gi; };
  auto locate = [&](int i) {
    int lo = 0, hi = a.batch;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if ((cu_in_lds ? s_cu[mid] : a.cu_tiles[mid]) <= i) lo = mid; else hi = mid;
    }
    Tile x;
    x.s = lo;
    x.row0 = (i - (cu_in_lds ? s_cu[lo] : a.cu_tiles[lo])) * a.tile_tokens;
    const int q = cu_in_lds ? s_cuq[lo + 1] - s_cuq[lo] : a.cu_q[lo + 1] - a.cu_q[lo];
    const int b = cu_in_lds ? s_beg[lo] : a.begin[lo];
    x.ntok = min(a.tile_tokens, q - x.row0);
    x.T = (b + x.row0 + x.ntok + a.ahead + kBN - 1) / kBN;   // room for the range to move up
    x.dmax = ((b + x.row0) / kBN) & ~1;
    x.pt = groups ? s_gp[lo] : 0;
    x.gm = groups && s_glead[lo] == lo ? s_gsize[lo] : 0;
    x.gi = groups && sliced ? s_common[lo] : x.gm;
    return x;
  };
  // (a batch of no more tiles than threads: a thread's tile is the same in every step)
  const bool one_each = total_tiles <= NT;
  Tile mine = {0, 0, 0, 0, 0, 0, 0, 0};
  if (one_each && t < total_tiles) mine = locate(t);
  auto tile = [&](int i) { return one_each ? mine : locate(i); };
  // own chunks of L tiles (L even) from the end of the group's prefix: [pt, pt+L), ...,
  // [pt+kL, T) with pt + kL <= dmax; the group's prefix itself in chunks of L
  auto own_splits = [&](const Tile& x, int L) { return L > 0 ? (x.dmax - x.pt) / L + 1 : 1; };
  auto grp_splits = [&](const Tile& x, int L) { return x.pt > 0 ? (L > 0 ? (x.pt + L - 1) / L : 1) : 0; };
  // arrival words per merge record and kv head: a tree over n chunks has up to n + log2(n) nodes; the
  // rows of the partial arrays they take
  auto arrive_words = [&](int L) { return 2 + (L > 0 ? s_maxcost / L + 16 : 16) / 32; };
  auto arrive_rows = [&](int L) { return (arrive_words(L) * a.hkv + a.hq - 1) / a.hq; };
  auto part_rows = [&](const Tile& x, int L, int arrive) {
    const int ns = own_splits(x, L);
    return (ns > 1 || x.pt > 0 ? ns * x.ntok + arrive : 0) + (x.gm ? grp_splits(x, L) * x.gm : 0);
  };
  auto total_part_rows = [&](int L) {   // block-wide
    long long rows = 0;
    const int arrive = arrive_rows(L);
    for (int i = t; i < total_tiles; i += NT) rows += part_rows(tile(i), L, arrive);
    return block_sum<NT>(rows, scan);
  };

  // 4. chunk length.  No cutting when the q tiles alone give the GPU kRoundsWanted rounds of
  //    work; otherwise a length that would make about kItemsPerSlot items per slot, never
  //    below the shortest piece of this kind of batch, doubled until the partial rows fit the
  //    workspace.
  int L = 0;
  if (kMayNarrow && narrow) {
    L = s_maxcost > kWholeNarrow ? (pieces + 1) & ~1 : s_maxcost;
  } else if (!wide && (int64_t)total_tiles * a.hkv < (int64_t)kRoundsWanted * a.slots) {
    long long cost = 0;
    for (int i = t; i < total_tiles; i += NT) {
      const Tile x = tile(i);
      cost += x.T - x.pt + (x.gi ? x.pt : 0);
    }
    cost = (long long)total_tiles * s_maxcost <= INT32_MAX ? block_sum_int<NT>((int)cost, scan)
                                                             : block_sum<NT>(cost, scan);
    const long long room = (long long)kItemsPerSlot * a.slots, heads = cost * a.hkv + room - 1;
    const long long want = heads <= INT32_MAX ? (int)heads / (int)room : heads / room;
    // short pieces: only if no sequence has two new tokens (as many q tiles as new tokens)
    int shortest = kMinChunkTiles;
    if (a.total_q <= total_tiles && want < kMinChunkTiles) {
      shortest = s_maxcost <= kMinChunkTilesShort * kMergeAhead ? kMinChunkTilesShort : kMinChunkTilesDecode;
      shortest = max(shortest, ((int)want + 1) & ~1);
      while (shortest < kMinChunkTiles &&
             !short_pieces_pay(a, shortest, s_maxcost, groups, total_tiles, (int)cost))
        shortest = min(2 * shortest, kMinChunkTiles);
    }
    L = want < shortest ? shortest : want > (1 << 28) ? (1 << 28) : (int)want;
    if (groups && sliced) {
      int longest = 0;
      for (int sq = 0; sq < a.batch; ++sq) longest = max(longest, s_gp[sq]);
      L = max(L, min((longest + kListedAhead - 2) / (kListedAhead - 1), kListedAhead));
    }
    L = (L + 1) & ~1;
  }
  while (L > 0) {
    if (L >= s_maxcost) { L = 0; break; }   // nothing is long enough to be cut
    // (each tile has at most s_maxcost / L + 1 chunks of its own, and as many of a prefix its tokens)
    const long long most = (long long)(groups ? 2 : 1) * (s_maxcost / L + 1) * a.total_q +
                           (long long)total_tiles * arrive_rows(L);
    if (most <= a.part_cap || total_part_rows(L) <= a.part_cap) break;
    L *= 2;
  }
  // without cuts the groups still need partial rows: no room, no groups
  if (L == 0 && groups && total_part_rows(0) > a.part_cap) {
    groups = false;
    mine.pt = mine.gm = mine.gi = 0;
  }

  int shift = 0;
  while ((s_maxcost >> shift) >= kBuckets) ++shift;
  auto bucket = [&](int len) { return kBuckets - 1 - (len >> shift); };
  // (a prefix's item of a whole q tile takes longer a tile than decode rows' items: those go first)
  auto group_bucket = [&](int len) { return bucket(sliced ? len : s_maxcost); };

  // 4b. remainder round.  Between one and kRoundsWanted rounds of uncut, similar items the last
  //     round is the problem: n items on S slots take ceil(n / S) rounds although the last one
  //     may hold few items.  The n mod S shortest items (they run last) are then cut into
  //     c = ceil(S / (n mod S)) chunks each, which fill that round with items 1/c as long.
  int tail_c = 0;
  {
    const int64_t n = (int64_t)total_tiles * a.hkv;
    const int rem = (int)(n % a.slots);
    const int rem_tiles = rem / a.hkv;
    const int c = rem > 0 ? min(8, (a.slots + rem - 1) / rem) : 0;
    if (L == 0 && !groups && !wide && !narrow && total_tiles <= kTailTilesMax && n >= a.slots &&
        n < (int64_t)kRoundsWanted * a.slots && rem_tiles >= 1 && 10 * rem <= 7 * a.slots && c >= 2 &&
        (int64_t)rem_tiles * (a.tile_tokens * c + arrive_rows(0)) <= a.part_cap) {
      if (t == 0) { s_tail_bucket = kBuckets; s_tail_take = 0; s_tail_taken = 0; }
      for (int i = t; i < total_tiles; i += NT) atomicAdd(&hist[bucket(locate(i).T)], 1);
      __syncthreads();
      // shortest first: walk the buckets from the last to the first until rem_tiles tiles are in
      constexpr int kPer = kBuckets / NT;
      int local[kPer], sum = 0;
      for (int i = 0; i < kPer; ++i) { local[i] = hist[kBuckets - 1 - (t * kPer + i)]; sum += local[i]; }
      int tot, before = block_exclusive_scan<NT>(sum, scan, &tot);
      for (int i = 0; i < kPer; ++i) {
        if (before < rem_tiles && before + local[i] >= rem_tiles) {
          s_tail_bucket = kBuckets - 1 - (t * kPer + i);
          s_tail_take = rem_tiles - before;
        }
        before += local[i];
      }
      __syncthreads();
      for (int i = t; i < total_tiles; i += NT) {
        const int bk = bucket(locate(i).T);
        s_tailflag[i] = bk > s_tail_bucket ||
                        (bk == s_tail_bucket && atomicAdd(&s_tail_taken, 1) < s_tail_take);
      }
      for (int i = t; i < kBuckets; i += NT) hist[i] = 0;
      __syncthreads();
      tail_c = c;
    }
  }
  // chunk length of q tile i: the batch's, or its own if it is cut for the remainder round
  auto chunk_len = [&](int i, const Tile& x) {
    if (tail_c == 0 || !s_tailflag[i]) return L;
    const int len = ((x.T + tail_c - 1) / tail_c + 1) & ~1;
    return max(len, kMinChunkTiles);
  };

  // 5. items and merge records: count per contiguous range of tiles, scan, histogram of costs
  const int tper = (total_tiles + NT - 1) / NT;
  const int i_lo = min(t * tper, total_tiles), i_hi = min(i_lo + tper, total_tiles);
  int n_items = 0, n_own = 0, n_grp = 0, n_merge = 0;
  for (int i = i_lo; i < i_hi; ++i) {
    const Tile x = tile(i);
    const int Li = chunk_len(i, x);
    const int ns = own_splits(x, Li), ng = x.gi ? grp_splits(x, Li) : 0;
    n_items += ns + ng;
    if (ns > 1 || x.pt > 0) { n_own += ns * x.ntok; ++n_merge; }
    n_grp += ng * x.gm;
    if (ns > 1) atomicAdd(&hist[bucket(Li)], ns - 1);
    atomicAdd(&hist[bucket(x.T - x.pt - (ns - 1) * Li)], 1);
    for (int c = 0; c < ng; ++c)
      atomicAdd(&hist[group_bucket(Li > 0 ? min(Li, x.pt - c * Li) : x.pt)], 1);
  }
  // 5b. the page ids: what step 2 requested, and the rest of the table.  The exact look: a wavefront takes four
  //     sequences per trip, four entries a lane, all of their loads in flight (the loop is bound by memory
  //     latency); entries beyond the first 256 of a sequence follow one sequence at a time.
  if (!suspect) {
#pragma unroll
    for (int k = 0; k < kFlatLoads; ++k) suspect |= bad_id(flat_ids[k]);
    if (!looked) look_at_rest();
  }
  if (__ballot(suspect) != 0 && (t & 63) == 0) s_suspect = 1;
  __syncthreads();
  if (ids_here && s_suspect) {
    const int lane4 = 4 * (t & 63);
    for (int s4 = (t >> 6) * 4; s4 < a.batch; s4 += (NT >> 6) * 4) {
      i32x4u pg[4];
      int need[4], p0[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int s = s4 + k;
        const int q = s < a.batch ? s_cuq[s + 1] - s_cuq[s] : 0;
        need[k] = q > 0 ? (s_beg[s] + q + a.ahead + kPage - 1) / kPage : 0;
        p0[k] = s < a.batch ? s_cup[s] : 0;
        pg[k] = i32x4u{0, 0, 0, 0};
        // (the last lane's four entries end with the last needed one: nothing beyond it is read)
        if (need[k] >= 4) {
          if (lane4 < need[k])
            pg[k] = *reinterpret_cast<const i32x4u*>(a.page_table + p0[k] + min(lane4, need[k] - 4));
        } else if ((t & 63) < need[k]) {
          pg[k][0] = a.page_table[p0[k] + (t & 63)];
        }
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (bad_id(pg[k])) err = 1;
        for (int i = 256 + lane4; i < need[k]; i += 256)
          if (bad_id(*reinterpret_cast<const i32x4u*>(a.page_table + p0[k] + min(i, need[k] - 4)))) err = 1;
      }
    }
  }
  if (__ballot(err != 0) != 0 && (t & 63) == 0) atomicOr(&s_err, 1);
  __syncthreads();
  constexpr int kPer = kBuckets / NT;
  int local[kPer], in_buckets = 0;
  for (int i = 0; i < kPer; ++i) { local[i] = hist[t * kPer + i]; in_buckets += local[i]; }
  int offs[5] = {n_items, n_own, n_grp, n_merge, in_buckets}, tots[5];
  block_exclusive_scan_n<NT>(offs, scan, tots);
  const int tot_items = tots[0], tot_own = tots[1], tot_grp = tots[2], tot_merge = tots[3];
  int item_off = offs[0], own_off = offs[1], grp_off = offs[2], merge_off = offs[3];
  for (int i = 0, off = offs[4]; i < kPer; ++i) { hist[t * kPer + i] = off; off += local[i]; }
  // a batch of no more tiles than threads: its items are written one a thread, not those of a tile one after
  // another (a load and a store behind it each), if a tile has more than four, or for decode steps' order (below).
  // Fewer are written sooner by the tile's thread (187 tiles of up to four pieces, one range, plan 13.7 -> 10.8 us) and lie
  // better: neighbours in the launch are of other tiles (13 rows beside a prefill of 2000 tokens, 32 / 8 heads, 48.9
  // us a layer, so 47.0; one range of 8 / 1 heads 109.2, 104.6).
  const bool by_tile = a.total_q <= total_tiles;
  const bool spread = one_each && tot_items > total_tiles && tot_items <= kSpreadItems &&
                      (by_tile || s_maxcost > 4 * L);
  if (spread && t < total_tiles) {
    s_first[t] = item_off;
    s_merge[t] = merge_off;
  }
  __syncthreads();
  if (s_err || tot_items > a.max_items || tot_own + tot_grp + (int64_t)tot_merge * arrive_rows(L) > a.part_cap ||
      tot_merge > a.max_merges) {   // a page id, or what cannot happen
    if (t == 0) refuse_plan(a.hdr);
    return;
  }
  // where each group's partial rows start (after all the tiles' own): its members need it
  if (groups) {
    int off = tot_own + grp_off;
    for (int i = i_lo; i < i_hi; ++i) {
      const Tile x = tile(i);
      if (x.gm) { s_gbase[x.s] = off; off += grp_splits(x, chunk_len(i, x)) * x.gm; }
    }
    __syncthreads();
  }
  for (int64_t i = t; i < (int64_t)tot_merge * a.hkv * arrive_words(L); i += NT)
    a.arrivals_end[-1 - i] = 0;   // nobody has arrived
  // 6. emit: counting sort of the items by cost (number of KV tiles), heaviest first
  //    Item k of tile x: of its own range's pieces, then of its prefix's; merge: the tile's record.
  //    (A piece takes a look at the table and the store of its record behind it, 0.3 us: one after the other
  //    by the tile's thread, 8 and 32 pieces of one decode row took 2.4 and 7.3 us, one a thread 1.1 and 1.2.
  //    With the page ids' look and without a sum that a bound replaces the plan of one row over 1000
  //    tokens takes 7.6 us instead of 10.0, over 8100 8.0 instead of 15.8, of 256 rows 14.4 instead of 19.4.)
  // Pieces of one length of decode steps lie tile by tile (by_tile), so that a row's last piece combines them while
  // others run (32 rows over 200..900 tokens, eight layers, 199 us, in the other order 206).  Else the first pieces of
  // all tiles lie ahead of their second ones, so that a compute unit's two workgroups differ (16 decode rows beside a
  // prefill of 600 tokens 145, so 137; 500 new tokens over 2500 184, so 178).
  struct Piece { int t0, t1, chunk; bool in_group; };
  auto piece = [&](const Tile& x, int Li, int k) {
    const int ns = own_splits(x, Li);
    const bool in_group = k >= ns;
    const int c = in_group ? k - ns : k, t0 = (in_group ? 0 : x.pt) + c * Li, end = in_group ? x.pt : x.T;
    return Piece{t0, Li > 0 && (in_group ? t0 + Li < end : k + 1 < ns) ? t0 + Li : end, c, in_group};
  };
  // its place in the list
  auto place_of = [&](const Piece& p) {
    return atomicAdd(&hist[p.in_group ? group_bucket(p.t1 - p.t0) : bucket(p.t1 - p.t0)], 1);
  };
  auto put_item = [&](const Tile& x, const Piece& p, bool merged, int merge, int at) {
    const int t0 = p.t0, t1 = p.t1, ntok = p.in_group ? x.gi : x.ntok;
    const int sq0 = cu_in_lds ? s_cuq[x.s] : a.cu_q[x.s];
    const int sq_len = (cu_in_lds ? s_cuq[x.s + 1] : a.cu_q[x.s + 1]) - sq0;
    const int sb = cu_in_lds ? s_beg[x.s] : a.begin[x.s];
    const int tab = cu_in_lds ? s_cup[x.s] : a.cu_pages[x.s];
    const int cap = (int)(((int64_t)sb + sq_len + a.ahead + kPage - 1) / kPage) - 1;   // validated above
    ItemRec it;
#pragma unroll
    for (int i = 0; i < 8; ++i) it.ids[i] = a.page_table[tab + min(4 * t0 + i, cap)];
    it.seq = x.s;
    it.row0 = p.in_group ? 0 : x.row0;
    it.chunk = merged ? p.chunk : -1;
    it.q_first = sq0 + it.row0;
    it.t0_ntok = (uint32_t)(t0 >> 1) | (uint32_t)(ntok - 1) << 24;
    // every tile of the item holds a validated entry, so the last one lies in tile t1 - 1 or beyond
    it.t1_flags = (uint32_t)t1 | (uint32_t)min(cap - 4 * (t1 - 1), 3) << 26 | (p.in_group ? kItemGroup : 0);
    it.table_off = tab;
    it.merge = merged ? merge : -1;
    a.items[at] = it;
  };
  for (int i = i_lo; i < i_hi; ++i) {
    const Tile x = tile(i);
    const int Li = chunk_len(i, x);
    const int ns = own_splits(x, Li), ng = grp_splits(x, Li);
    const int merge = merge_off, n = ns + (x.gi ? ng : 0);
    const bool merged = ns > 1 || x.pt > 0;
    if (merged) {
      MergeRec m;
      m.q_row = (cu_in_lds ? s_cuq[x.s] : a.cu_q[x.s]) + x.row0;
      m.ntok = x.ntok;
      m.nsplit = ns;
      m.part = own_off;
      m.g_nsplit = ng;
      m.g_part = x.pt > 0 ? s_gbase[s_glead[x.s]] : 0;
      m.g_stride = x.pt > 0 ? s_gsize[s_glead[x.s]] : 0;
      m.g_off = x.pt > 0 ? s_cuq[x.s] - s_cuq[s_glead[x.s]] : 0;
      a.merges[merge_off++] = m;
      own_off += ns * x.ntok;
    }
    if (spread) {
#pragma unroll 4
      for (int k = 0; k < n; ++k) {
        if (!by_tile) s_place[item_off + k] = (uint16_t)place_of(piece(x, Li, k));
        s_owner[item_off + k] = (uint16_t)t;
      }
    } else {
      for (int k = 0; k < n; ++k) {
        const Piece p = piece(x, Li, k);
        put_item(x, p, merged, merge, place_of(p));
      }
    }
  }
  if (spread) {
    __syncthreads();
    for (int j = t; j < tot_items; j += NT) {
      const int i = s_owner[j];
      const Tile x = locate(i);
      const int Li = chunk_len(i, x);
      const Piece p = piece(x, Li, j - s_first[i]);
      put_item(x, p, own_splits(x, Li) > 1 || x.pt > 0, s_merge[i], by_tile ? place_of(p) : s_place[j]);
    }
  }
  if (t == 0) {
    a.hdr->err = MC_OK;
    a.hdr->heads = head_counts(a.hkv, a.hq / a.hkv);
    a.hdr->num_items = tot_items;
    a.hdr->num_merges = tot_merge;
    a.hdr->chunk_tiles = L;
    a.hdr->tile_tokens = a.tile_tokens;
    a.hdr->batch = a.batch;
    a.hdr->total_q = a.total_q;
    a.hdr->num_groups_rows = tot_grp;
    a.hdr->tail_chunks = tail_c;
    a.hdr->arrive_words = arrive_words(L);
    a.hdr->magic = kPlanMagic;
  }
}

// ----------------------------------------------------------- attention ------
template <typename T> struct Mfma;
template <> struct Mfma<_Float16> {
  typedef f16x8 vec8;
  static __device__ __forceinline__ f32x16 run(vec8 a, vec8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ f32x4 run16(vec8 a, vec8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
  }
  // the 32x32x16 one with its result pinned to vector registers (see attn_kernel: with
  // two row blocks the allocator would otherwise park the scores in accumulation registers,
  // which the softmax's vector instructions cannot read)
  static __device__ __forceinline__ void run_v0(vec8 a, vec8 b, f32x16& c) {
    asm("v_mfma_f32_32x32x16_f16 %0, %1, %2, 0" : "=v"(c) : "v"(a), "v"(b));
  }
  static __device__ __forceinline__ void run_v(vec8 a, vec8 b, f32x16& c) {
    asm("v_mfma_f32_32x32x16_f16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
  }
  static __device__ __forceinline__ uint32_t pack2(float x, float y) {
    typedef _Float16 h2 __attribute__((ext_vector_type(2)));
    h2 v;
    v[0] = (_Float16)x;
    v[1] = (_Float16)y;
    return __builtin_bit_cast(uint32_t, v);
  }
};
template <> struct Mfma<__bf16> {
  typedef bf16x8 vec8;
  static __device__ __forceinline__ f32x16 run(vec8 a, vec8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ f32x4 run16(vec8 a, vec8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ void run_v0(vec8 a, vec8 b, f32x16& c) {
    asm("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=v"(c) : "v"(a), "v"(b));
  }
  static __device__ __forceinline__ void run_v(vec8 a, vec8 b, f32x16& c) {
    asm("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
  }
  static __device__ __forceinline__ uint32_t pack2(float x, float y) {
    typedef __bf16 b2 __attribute__((ext_vector_type(2)));
    b2 v;
    v[0] = (__bf16)x;
    v[1] = (__bf16)y;
    return __builtin_bit_cast(uint32_t, v);
  }
};

struct AttnArgs {
  const char* pool_layer;  // pool base + layer offset
  const char* q;
  char* out;
  float* lse;
  const int32_t* begin;
  const int32_t* page_table;
  const PlanHeader* hdr;
  const ItemRec* items;
  const MergeRec* merges;
  float* part_lse;         // of every partial row (see MergeRec); the arrival words at its end
  float* part_o;           // [partial row][128]
  int32_t num_pages, hkv, hq, batch, total_q;
  int32_t units;           // compute units
  int32_t part_cap;        // rows of the partial arrays
  int32_t behind;          // what merge_kernel combines (see MergeRec): kGroupsBehind, kTreesBehind
  float scale, scale_log2;  // softmax scale, and scale * log2(e)
};

typedef s16x4 __attribute__((address_space(3))) * lds_s16x4_ptr;
typedef __attribute__((address_space(3))) void* lds_void_ptr;
// Read-only metadata is addressed through the constant address space so that wave-uniform
// reads stay scalar loads (no vector-memory counter involved) even after LDS copies and stores.
typedef const __attribute__((address_space(4))) int32_t* const_i32_ptr;

constexpr int kTileBytes = kBN * kRowBytes;   // one K or V tile in LDS: 16 KiB

// The fixed-reference pass (see attn_kernel's run_pass) is tried first where P keeps fp32's
// exponent range.  fp16 holds p only up to 2^16: there the reference must follow the row max.
template <typename T> constexpr bool kTryFixedRef = false;
#ifndef MC_NO_FIXED_REF
template <> constexpr bool kTryFixedRef<__bf16> = true;
#endif
// A row sum below this proves that no exponential of the pass overflowed (every p is at most
// the sum) and that P fitted its 2-byte type; the O accumulators are checked for finiteness
// separately.  Reached only when a score exceeds the first half tile's maximum by more than
// 60 in the exp2 domain (about 41 in natural units).
constexpr float kFixedRefSumLimit = 0x1p+60f;
// register pairs of S(h) whose exponentials run in phase 2 of a fixed-reference half step
#ifndef MC_PAIRS_LATE
#define MC_PAIRS_LATE 4
#endif
constexpr int kPairsLate = MC_PAIRS_LATE;
// MFMA slot (0..15 of a half step) after which the first of a tile's eight copies is issued in
// the main loop; one more follows after each later slot
#ifndef MC_COPY_SLOT0
#define MC_COPY_SLOT0 4
#endif
constexpr int kCopySlot0 = MC_COPY_SLOT0;
static_assert(kCopySlot0 >= 1 && kCopySlot0 <= 8, "eight copy slots and one for the addresses before them");
static_assert(kPairsLate >= 0 && kPairsLate <= 4, "operand words 4..7 are read from phase 2's step 4 on");

__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return (uint32_t)(size_t)(lds_void_ptr)(p);
}

// Asynchronous 16-byte-per-lane copy from global memory straight into LDS: lane L's bytes
// land at lds_base + 16 L.  base and lds_base are wave-uniform.  Issued as inline assembly so
// that the compiler does not serialise it against later LDS reads of OTHER buffers; completion
// is awaited explicitly (s_waitcnt vmcnt(0)) before the workgroup barrier that publishes it.
__device__ __forceinline__ void copy16_to_lds(const char* base, uint32_t lane_off,
                                              uint32_t lds_base) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :: "v"(lane_off), "s"(base), "s"(lds_base) : "memory", "m0");
}

// ---- partial rows ------------------------------------------------------------------------
// They are written by one workgroup and read by another of the same launch, on any XCD: through
// buffer instructions of device scope (sc1), which write to and read from the level all XCDs
// share, so that no L2 has to be written back or invalidated as a whole.  Rows that merge_kernel
// reads go by plain ones (kLaunchScope): the launch's end makes them visible, and an L2 gathers the 16
// bytes a lane that a row by row store of 32 rows is made of.
typedef __amdgpu_buffer_rsrc_t buffer_rsrc;
constexpr int kDeviceScope = 16, kLaunchScope = 0;          // sc1, none
__device__ __forceinline__ buffer_rsrc make_rsrc(void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(p, 0, bytes, 0x00020000);   // raw, 32-bit; bounds checked
}
template <int kScope>
__device__ __forceinline__ void store_part(buffer_rsrc r, uint32_t off, f32x4 v) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), r, off, 0, kScope);
}
template <int kScope>
__device__ __forceinline__ void store_part(buffer_rsrc r, uint32_t off, float v) {
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, off, 0, kScope);
}
template <int kScope>
__device__ __forceinline__ f32x4 load_part4(buffer_rsrc r, uint32_t off) {
  return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, kScope));
}
template <int kScope>
__device__ __forceinline__ float load_part(buffer_rsrc r, uint32_t off) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, kScope));
}

// Chunks of a tile's own that a merge record's last step combines (a tree's count as one).
template <int G>
__device__ __forceinline__ int own_chunks(int flat, bool trees, int nsplit, int ntok) {
  return ntok * G <= flat || !trees ? nsplit : 1;
}

// What a workgroup was the last to arrive at, in LDS (the tiles are consumed): the merge records, the
// first token of each among all whose rows are to be combined, and the record a token belongs to.
struct MergeList {
  int32_t rec[kBM][8];             // MergeRec
  int32_t first[kBM], rec_of[2 * kBM];
};
static_assert(sizeof(MergeList) <= 4 * kTileBytes, "the list takes the tiles' LDS");

// One more chunk of a row (LSE lse) beside those summed so far (their maximum mx, their weights' sum
// den): the factors of both.  Every place that sums chunks does it by this step, chunk after chunk in
// their order, so that the result does not depend on the place.  A chunk without a key (LSE -inf) has
// no weight, and no maximum; one whose LSE is not a number has a weight that is none either, which den
// and the row then are.  den is 0 until a chunk with a key has come.
__device__ __forceinline__ void chunk_step(float lse, float& mx, float& den, float& f_old, float& f_new) {
  const float m = fmaxf(mx, lse);
  f_old = m > -INFINITY ? __expf(mx - m) : 1.f;
  f_new = lse != -INFINITY ? __expf(lse - m) : 0.f;
  mx = m;
  den = __builtin_fmaf(den, f_old, f_new);
}

// One kv head's rows of `tokens` tokens from their chunks: with L_c the chunk LSEs, LSE = log sum_c
// exp(L_c) and O = sum_c exp(L_c - LSE) O_c, chunks in order: those of the group's prefix, then the tile's
// own.  record(i, first) gives the merge record of token i and the first token of that record.  Of `blocks`
// workgroups that share the rows this is number `block`; trees: chunks of many rows have gone up a tree.
// A chain of memory round trips and little else, run once by code that is not in the instruction
// cache: half a wavefront takes a row, 16 bytes a lane; every lane forms the row's weights by itself
// from LSEs it reads beside the rows (no exchange, no barrier); kRows rows x kChunks chunks are in
// flight, and nothing but the loop stands under a condition.
template <typename T, int G, int kScope, int kRows, int kChunks, typename Record>
__device__ __forceinline__ void merge_rows(const AttnArgs& a, buffer_rsrc rs_o, buffer_rsrc rs_lse,
                                           int hk, int tokens, int flat, bool trees, int block, int blocks,
                                           Record&& record) {
  const int rows = tokens * G, piece = threadIdx.x & 31;
  for (int r0 = (threadIdx.x >> 5) + block * kRows * (kThreads / 32); r0 < rows;
       r0 += blocks * kRows * (kThreads / 32)) {
    // per row: chunks, the prefix's among them, partial row and byte of this lane's piece in the first
    // chunk, the same from one chunk to the next
    int nch[kRows], g_nsplit[kRows], out_row[kRows];
    uint32_t g_row[kRows], g_byte[kRows], g_step[kRows], own_row[kRows], own_byte[kRows], own_step[kRows];
    float mx[kRows], den[kRows];
    f32x4 acc[kRows];
    int nmax = 0;
#pragma unroll
    for (int u = 0; u < kRows; ++u) {
      const int r = min(r0 + u * (kThreads / 32), rows - 1), i = r / G;
      int first;
      const auto m = record(i, first);
      const int tt = i - first;
      // row r of the chunk whose rows, of_rows of them, start at row0
      auto place = [&](uint32_t row0, int r, int of_rows) __attribute__((always_inline)) {
        return row0 * 512u + (of_rows <= flat || !trees
                                  ? r * 512u + piece * 16u
                                  : (piece >> 1) * of_rows * 32u + r * 32u + (piece & 1) * 16u);
      };
      g_nsplit[u] = m[4];
      nch[u] = own_chunks<G>(flat, trees, m[2], m[1]) + m[4];
      const uint32_t g0 = m[5] * a.hq + hk * m[6] * G, own0 = m[3] * a.hq + hk * m[1] * G;
      const int g_r = (m[7] + tt) * G + r % G, own_r = tt * G + r % G;
      g_row[u] = g0 + g_r;
      g_byte[u] = (g0 + g_r) * 512u + piece * 16u;
      g_step[u] = m[6] * a.hq;
      own_row[u] = own0 + own_r;
      own_byte[u] = place(own0, own_r, m[1] * G);
      own_step[u] = m[1] * a.hq;
      out_row[u] = (m[0] + tt) * a.hq + hk * G + r % G;
      mx[u] = -INFINITY;
      den[u] = 0.f;
      acc[u] = f32x4{0.f, 0.f, 0.f, 0.f};
      nmax = max(nmax, nch[u]);
    }
    for (int c0 = 0; c0 < nmax; c0 += kChunks) {
      f32x4 o[kRows][kChunks];
      float lse[kRows][kChunks];
#pragma unroll
      for (int u = 0; u < kRows; ++u)
#pragma unroll
        for (int k = 0; k < kChunks; ++k) {
          const int c = min(c0 + k, nch[u] - 1);
          const bool in_group = c < g_nsplit[u];
          const uint32_t on = (in_group ? c : c - g_nsplit[u]) * (in_group ? g_step[u] : own_step[u]);
          lse[u][k] = load_part<kScope>(rs_lse, ((in_group ? g_row[u] : own_row[u]) + on) * 4u);
          o[u][k] = load_part4<kScope>(rs_o, (in_group ? g_byte[u] : own_byte[u]) + on * 512u);
        }
#pragma unroll
      for (int u = 0; u < kRows; ++u)
#pragma unroll
        for (int k = 0; k < kChunks; ++k) {
          const float l = c0 + k < nch[u] ? lse[u][k] : -INFINITY;
          float f_old, f_new;
          chunk_step(l, mx[u], den[u], f_old, f_new);
          // A chunk without a key is left out, not weighed by 0: one that was not computed left in its
          // rows what the memory held before, which may be NaN.
#pragma unroll
          for (int j = 0; j < 4; ++j)
            acc[u][j] = __builtin_fmaf(l != -INFINITY ? o[u][k][j] : 0.f, f_new, acc[u][j] * f_old);
        }
    }
#pragma unroll
    for (int u = 0; u < kRows; ++u) {
      // (no chunk of the row was computed: nothing is written)
      if (r0 + u * (kThreads / 32) >= rows || den[u] == 0.f) continue;
      const float inv = 1.f / den[u];
      u32x2 v;
      v[0] = Mfma<T>::pack2(acc[u][0] * inv, acc[u][1] * inv);
      v[1] = Mfma<T>::pack2(acc[u][2] * inv, acc[u][3] * inv);
      *reinterpret_cast<u32x2*>(a.out + (int64_t)out_row[u] * kRowBytes + piece * 8) = v;
      if (piece == 0) a.lse[out_row[u]] = mx[u] + __logf(den[u]);
    }
  }
}

// LDS tile: 64 rows (keys) x 256 B.  16-byte chunk c of row r sits at chunk position
//   K: c ^ (r & 15)        -> 16 lanes reading one chunk of 16 consecutive rows hit 16 positions
//   V: c ^ ((r & 3) << 2)  -> a transposing read of 4 consecutive rows x 64 B hits 16 positions
__device__ __forceinline__ int k_swz(int row, int chunk) { return row * kRowBytes + ((chunk ^ (row & 15)) << 4); }
__device__ __forceinline__ int v_swz(int row, int chunk) { return row * kRowBytes + ((chunk ^ ((row & 3) << 2)) << 4); }

// max of three floats in one instruction (written as assembly: through fmaxf every score would
// first pass a NaN-quieting instruction of its own).  The compiler does not see what an assembly
// statement reads, so it inserts none of the wait states a vector instruction needs before it
// may read the registers an MFMA is still writing: the first read of a fresh MFMA result goes
// through fmaxf, which the compiler does protect, and only the later ones through this.
__device__ __forceinline__ float max3(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

// ---- items of few rows (decode steps) ----------------------------------------------------
// What an item needs of its record.
struct Item {
  int t0, t1, chunk, q_first, ntok, table_off, pidx_cap, merge, n_rec;   // n_rec: merge records there are
  int behind;
  bool group;
};

// The first of the partial rows of a chunk and kv head that an item writes (m: its merge record, of a
// group its first member's).
template <int G>
__device__ __forceinline__ uint32_t first_part_row(const AttnArgs& a, const Item& it, int hk, const i32x8& m) {
  return it.group ? (m[5] + it.chunk * m[6]) * a.hq + (hk * m[6] + m[7]) * G
                  : (m[3] + it.chunk * m[1]) * a.hq + hk * m[1] * G;
}

// Whether a chunk that is no tree's is combined inside this launch; else merge_kernel does it behind it.
template <int G, int kFlat>
__device__ __forceinline__ bool combined_here(const Item& it, const i32x8& m) {
  return it.group || m[4] > 0 ? !(it.behind & kGroupsBehind) : it.ntok * G <= kFlat;
}

// Counts written rows - a chunk of few rows, a chunk of a prefix (at every member's record), or a tree's
// result - and, if they were the last there, combines the record's chunks.  s_last: 0, and published;
// list: free LDS.
template <typename T, int G, int kFlat, int kRows>
__device__ __forceinline__ void arrive(const AttnArgs& a, const Item& it, int hk, buffer_rsrc rs_o,
                                       buffer_rsrc rs_lse, const i32x8& m, int words, int& s_last,
                                       MergeList& list) {
  const int tid = threadIdx.x;
  const bool listed = it.group || it.ntok * G > kFlat;
  uint32_t* arrivals = reinterpret_cast<uint32_t*>(a.part_lse) + (int64_t)a.part_cap * a.hq - 1;
  i32x8 mr = m;
  if (it.group) mr = *reinterpret_cast<const i32x8*>(a.merges + min(it.merge + tid, it.n_rec - 1));
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wavefront's rows have been written
  __syncthreads();
  // records of this item: one, or the group's members' (their tokens follow one another)
  if (tid < (it.group ? it.ntok : 1) && it.merge + tid < it.n_rec && mr[0] < it.q_first + it.ntok) {
    const int n = own_chunks<G>(kFlat, true, mr[2], mr[1]) + mr[4];
    if (atomicInc(arrivals - ((int64_t)(it.merge + tid) * a.hkv + hk) * words, n - 1) == (unsigned)n - 1) {
      const int at = atomicAdd(&s_last, mr[1]);
      if (listed) {
        *reinterpret_cast<i32x8*>(list.rec[tid]) = mr;
        list.first[tid] = at;
        if (it.group)
          for (int i = 0; i < mr[1]; ++i) list.rec_of[at + i] = tid;
      }
    }
  }
  if (listed && !it.group && tid < it.ntok) list.rec_of[tid] = 0;
  __syncthreads();
  const int tokens = __builtin_amdgcn_readfirstlane(s_last);
  if (tokens == 0) return;
  if (listed)
    merge_rows<T, G, kDeviceScope, 2, kListedAhead>(
        a, rs_o, rs_lse, hk, tokens, kFlat, true, 0, 1, [&](int i, int& first) __attribute__((always_inline)) {
      const int k = list.rec_of[i];
      first = list.first[k];
      return *reinterpret_cast<const i32x8*>(list.rec[k]);
    });
  else
    merge_rows<T, G, kDeviceScope, kRows, kMergeAhead>(
        a, rs_o, rs_lse, hk, tokens, kFlat, true, 0, 1, [&](int, int& first) __attribute__((always_inline)) { first = 0; return m; });
}

// max or sum over the four lanes l, l ^ 16, l ^ 32, l ^ 48: a swap of the wavefront's halves, then one
// of its odd with its even rows of 16 lanes, each given the value in both operands (see
// max_across_halves below for the assembly)
template <typename Op>
__device__ __forceinline__ float across_rows(float x, Op&& op) {
  uint32_t lo = __builtin_bit_cast(uint32_t, x), hi = lo;
  asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(lo), "+v"(hi));
  lo = hi = __builtin_bit_cast(uint32_t, op(__builtin_bit_cast(float, lo), __builtin_bit_cast(float, hi)));
  asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(lo), "+v"(hi));
  return op(__builtin_bit_cast(float, lo), __builtin_bit_cast(float, hi));
}

// An item of at most 16 rows, or of two blocks of 16 which share every K and V fragment (kRB = 2).  All four
// wavefronts hold those rows and take half tiles (32 keys, 2 pages) in turn, each by itself: K straight into
// registers, V through its own 16 KiB of LDS, no barrier until their sums are put together at the end.
// v_mfma_f32_16x16x32: S^T = K Q^T (A = 16
// keys, lane l: key l % 16, d 8 (l / 16) ..), a lane then has one row (l % 16) and 8 of the 32 keys;
// O^T += V^T P^T with P^T straight from S^T: operand slot 8 g + j is key 4 g + j of the first 16 keys
// (j < 4) or of the second, for both operands (g = l / 16).
// Decode steps are bound by memory: on few rows by the latency of the requests that follow one
// another, else by the reads themselves.  Walked by one wavefront of four, as items of more rows are
// (the other three without a row), a piece of two tiles took 5.0 us from the first instruction to the
// vote at its end, three requests behind the record; here one, the first half tile of every wavefront.
// K and V take turns, 8 KiB in flight for each of a compute unit's eight wavefronts: the next half tile's V
// is requested and waited for when K has come, then S is formed and the next K requested, which is under way
// while the softmax and P V run.  More in flight is slower where the reads are the bound: with the next V
// under way beside K (one wait a half tile, behind the next V's request), or beside S and the next K (no
// second wait), us a pass of 43 rows over 166..1205 keys, 16 / 8 heads, four layers 143.9 -> 147.2, 148.4;
// of 64 forks of a 2048-token prompt, 32 / 8, four layers 196.1 -> 200.3, 200.1; of 64 rows over 1024..4096
// beside a prefill, two layers 328 -> 329, 336; of eight rows over 1024..4096, 64 / 8, eight layers 207.0 ->
// 205.0, 205.4.
// beside: a workgroup a compute unit at most, as in plans of narrow q tiles, their keys in the L2s: bound by latency, so
// V is requested beside K there (256 tokens over 256, 8 / 8 heads, 11.8 -> 11.3 us a layer; 128 over 1024, 32 / 8, 19.5 ->
// 19.0; 16 over 300, 8 / 8, a whole tile, 11.9 -> 11.5).  Only in the launch that may have narrow tiles (kNarrow), and not for
// the decode rows of plans of more items, which it runs as well (eight rows over 16000 beside 128 new tokens, 8 / 1 heads,
// 31.1 us a layer, 28.4 with V ahead).
// A layer (append and attention) of one row over 1000 keys, 32 / 8 heads, 12.9 -> 10.5 us; of eight rows
// over 1024..4096, 64 / 8 heads, 27.7 -> 25.5; 256 rows, bound by the reads, the same.
template <typename T, int G, int kRB, bool kNarrow>
__device__ __forceinline__ void few_rows_item(const AttnArgs& a, const Item& it, int hk, int b, int row0,
                                              const i32x8& ids, char* lds, float* stat, int& s_last,
                                              bool beside) {
  typedef typename Mfma<T>::vec8 vec8;
  constexpr int kHalf = kBN / 2, kHalfBytes = kHalf * kRowBytes;
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g4 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rows = it.ntok * G;
  const uint32_t lds_own = lds_addr(lds) + wave * (2 * kHalfBytes);
  const char* pool_k = a.pool_layer + (int64_t)hk * kHeadPageBytes;
  const uint32_t page_blocks = 2u * a.hkv;                     // 4 KiB blocks per page
  auto page_base = [&](int32_t pg) __attribute__((always_inline)) {
    pg = min(max(pg, 0), a.num_pages - 1);         // checked by the plan; stay in bounds anyway
    return pool_k + ((uint64_t)((uint32_t)pg * page_blocks) << 12);
  };
  // K: key l16 of each page, chunks 4 kk + g4; V: 4 rows an instruction, swizzled as tiles are
  const uint32_t k_off = l16 * kRowBytes + g4 * 16;
  const uint32_t v_off = g4 * kRowBytes + ((l16 ^ (g4 << 2)) << 4) + (uint32_t)a.hkv * kHeadPageBytes;
  vec8 kf[2][4], q[kRB][4];
  auto request_v = [&](int32_t id0, int32_t id1, int buf) __attribute__((always_inline)) {
    const char* page[2] = {page_base(id0), page_base(id1)};
#pragma unroll
    for (int i = 0; i < 8; ++i)
      copy16_to_lds(page[i >> 2] + (i & 3) * 1024, v_off, lds_own + buf * kHalfBytes + i * 1024);
  };
  auto request_k = [&](int32_t id0, int32_t id1) __attribute__((always_inline)) {
    const char* page[2] = {page_base(id0), page_base(id1)};
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
        kf[p][kk] = __builtin_bit_cast(vec8, *reinterpret_cast<const u32x4*>(page[p] + k_off + kk * 64));
  };
  // page ids of the wavefront's half tile h (the first: in the record); clamped to validated entries
  const const_i32_ptr table = (const_i32_ptr)(a.page_table + it.table_off);
  auto id_of = [&](int h, int p) __attribute__((always_inline)) { return table[min(2 * h + p, it.pidx_cap)]; };
  int h = 2 * it.t0 + wave;
  int32_t next0 = id_of(h + 4, 0), next1 = id_of(h + 4, 1);
  if (h < 2 * it.t1) {
    const int32_t id0 = wave == 0 ? ids[0] : wave == 1 ? ids[2] : wave == 2 ? ids[4] : ids[6];
    const int32_t id1 = wave == 0 ? ids[1] : wave == 1 ? ids[3] : wave == 2 ? ids[5] : ids[7];
    request_v(id0, id1, 0);
    request_k(id0, id1);
  }
  // this lane's row of each block (one that does not exist reads the last one's q)
  int tt[kRB];
#pragma unroll
  for (int rb = 0; rb < kRB; ++rb) {
    const int my_row = min(16 * rb + l16, rows - 1);
    tt[rb] = my_row / G;
    const char* q_row = a.q + ((int64_t)(it.q_first + tt[rb]) * a.hq + hk * G + my_row % G) * kRowBytes;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
      q[rb][kk] = __builtin_bit_cast(vec8, *reinterpret_cast<const u32x4*>(q_row + kk * 64 + g4 * 16));
  }

  // positions: as in attn_kernel
  const int first_pos = it.group ? it.t1 * kBN : b + row0;
  const int kv_len = min(first_pos + it.ntok, it.t1 * kBN);
  const bool fits = b >= 0 && kv_len > kBN * it.t0;
  const int n_halves = fits ? (kv_len + kHalf - 1) / kHalf : 0;
  const int n_full = (first_pos + 1) / kHalf;
  const float c2 = a.scale_log2;

  f32x4 o[kRB][8];
  float m_run[kRB], l_run[kRB];     // the row's running maximum (raw); this lane's part of its sum
#pragma unroll
  for (int rb = 0; rb < kRB; ++rb) {
#pragma unroll
    for (int i = 0; i < 8; ++i) o[rb][i] = f32x4{0.f, 0.f, 0.f, 0.f};
    m_run[rb] = -INFINITY;
    l_run[rb] = 0.f;
  }
  int buf = 0;
  for (; h < n_halves; h += 4, buf ^= 1) {
    const bool more = h + 4 < n_halves;
    if constexpr (kNarrow) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the other V buffer has been read
    if (!beside) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      if (more) request_v(next0, next1, buf ^ 1);
    }
    // (K and q pass through the wait: the compiler, which counts its own loads but not the copies, would
    // else wait for them once more ahead of S)
    asm volatile("s_waitcnt vmcnt(0)"
                 : "+v"(kf[0][0]), "+v"(kf[0][1]), "+v"(kf[0][2]), "+v"(kf[0][3]), "+v"(kf[1][0]), "+v"(kf[1][1]),
                   "+v"(kf[1][2]), "+v"(kf[1][3]), "+v"(q[0][0]), "+v"(q[0][1]), "+v"(q[0][2]), "+v"(q[0][3]),
                   "+v"(q[kRB - 1][0]), "+v"(q[kRB - 1][1]), "+v"(q[kRB - 1][2]), "+v"(q[kRB - 1][3])
                 :
                 : "memory");
    f32x4 s[kRB][2];
#pragma unroll
    for (int rb = 0; rb < kRB; ++rb) s[rb][0] = s[rb][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
      for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int rb = 0; rb < kRB; ++rb) s[rb][p] = Mfma<T>::run16(kf[p][kk], q[rb][kk], s[rb][p]);
    if (more) {
      if (beside) request_v(next0, next1, buf ^ 1);
      request_k(next0, next1);
      next0 = id_of(h + 8, 0);
      next1 = id_of(h + 8, 1);
    }
    const uint32_t v_buf = lds_own + buf * kHalfBytes;
    if (kv_len < (h + 1) * kHalf) {      // V rows of keys past the range: 0 x NaN would poison O
      const int valid = kv_len - h * kHalf;
      const u32x4 zero = {0, 0, 0, 0};
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (4 * i + g4 >= valid)
          *reinterpret_cast<u32x4 __attribute__((address_space(3)))*>((size_t)(v_buf + i * 1024 + lane * 16)) = zero;
    }
    float alpha[kRB];
    u32x4 pw[kRB];
#pragma unroll
    for (int rb = 0; rb < kRB; ++rb) {
      if (h >= n_full) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
          if (h * kHalf + 16 * (i >> 2) + 4 * g4 + (i & 3) > first_pos + tt[rb]) s[rb][i >> 2][i & 3] = -INFINITY;
      }
      const f32x4 &s0 = s[rb][0], &s1 = s[rb][1];
      float mx = fmaxf(fmaxf(fmaxf(s0[0], s0[1]), fmaxf(s0[2], s0[3])), fmaxf(fmaxf(s1[0], s1[1]), fmaxf(s1[2], s1[3])));
      mx = fmaxf(m_run[rb], across_rows(mx, [](float x, float y) { return fmaxf(x, y); }));
      const float ref = mx > -INFINITY ? mx : 0.f, mc2 = ref * c2;      // (no key seen yet: no maximum)
      alpha[rb] = __builtin_amdgcn_exp2f((m_run[rb] - ref) * c2);
      m_run[rb] = mx;
      float p[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) p[i] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[rb][i >> 2][i & 3], c2, -mc2));
      l_run[rb] = __builtin_fmaf(l_run[rb], alpha[rb],
                                 ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7])));
      pw[rb] = u32x4{Mfma<T>::pack2(p[0], p[1]), Mfma<T>::pack2(p[2], p[3]), Mfma<T>::pack2(p[4], p[5]),
                     Mfma<T>::pack2(p[6], p[7])};
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int key = 4 * g4 + (l16 >> 2), at = 2 * i + ((l16 & 3) >> 1), sub = (l16 & 1) * 8;
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(size_t)(v_buf + v_swz(key, at) + sub));
      const s16x4 hi =
          __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(size_t)(v_buf + v_swz(key + 16, at) + sub));
      const vec8 vf = __builtin_bit_cast(vec8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
      for (int rb = 0; rb < kRB; ++rb) {
        o[rb][i] *= alpha[rb];
        o[rb][i] = Mfma<T>::run16(vf, __builtin_bit_cast(vec8, pw[rb]), o[rb][i]);
      }
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (a half tile past the range may be under way)
  if (!fits && it.chunk < 0) return;

  // ---- the four wavefronts' sums: O by rows of 32 pieces of 16 bytes (piece 4 i + g4: d = 16 i + 4 g4
  //      + {0..3}; the swizzle spreads the rows over the banks), each in its own LDS
  constexpr int kRows = 16 * kRB;
#pragma unroll
  for (int rb = 0; rb < kRB; ++rb) {
    const int r = 16 * rb + l16;
    l_run[rb] = across_rows(l_run[rb], [](float x, float y) { return x + y; });
    if (r < rows) {
#pragma unroll
      for (int i = 0; i < 8; ++i)
        *reinterpret_cast<f32x4*>(lds + wave * (2 * kHalfBytes) + r * 512 + (((4 * i + g4) ^ r) << 4)) = o[rb][i];
    }
    if (lane < 16) {
      stat[wave * kRows + r] = m_run[rb];
      stat[(4 + wave) * kRows + r] = l_run[rb];
    }
  }
  __syncthreads();
  const buffer_rsrc rs_o = make_rsrc(a.part_o, (uint32_t)a.part_cap * a.hq * 512u);
  const buffer_rsrc rs_lse = make_rsrc(a.part_lse, (uint32_t)a.part_cap * a.hq * 4u);
  i32x8 m = {0, 0, 0, 0, 0, 0, 0, 0};
  int words = 0;
  constexpr int kFlat = kNarrow ? kNarrowRows : kFlatRows;
  const bool chunk = it.chunk >= 0;
  if (chunk) {
    m = *(const __attribute__((address_space(4))) i32x8*)(a.merges + it.merge);
    words = ((const_i32_ptr)a.hdr)[10];
  }
  const uint32_t part0 = first_part_row<G>(a, it, hk, m);
  for (int r = tid >> 5; r < rows; r += kThreads / 32) {
    const int piece = tid & 31;
    float mx = -INFINITY;
#pragma unroll
    for (int w = 0; w < 4; ++w) mx = fmaxf(mx, stat[w * kRows + r]);
    const float ref = mx > -INFINITY ? mx : 0.f;
    float sum = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float f = __builtin_amdgcn_exp2f((stat[w * kRows + r] - ref) * c2);
      sum = __builtin_fmaf(stat[(4 + w) * kRows + r], f, sum);
      acc += f * *reinterpret_cast<const f32x4*>(lds + w * (2 * kHalfBytes) + r * 512 + ((piece ^ r) << 4));
    }
    const float inv = fits ? 1.f / sum : 0.f, lse = fits ? mx * a.scale + __logf(sum) : -INFINITY;
    acc *= inv;
    if (chunk && !combined_here<G, kFlat>(it, m)) {
      store_part<kLaunchScope>(rs_o, (part0 + r) * 512u + piece * 16u, acc);
      if (piece == 0) store_part<kLaunchScope>(rs_lse, (part0 + r) * 4u, lse);
    } else if (chunk) {
      store_part<kDeviceScope>(rs_o, (part0 + r) * 512u + piece * 16u, acc);
      if (piece == 0) store_part<kDeviceScope>(rs_lse, (part0 + r) * 4u, lse);
    } else {
      const int64_t out_row = (int64_t)(it.q_first + r / G) * a.hq + hk * G + r % G;
      const u32x2 v = {Mfma<T>::pack2(acc[0], acc[1]), Mfma<T>::pack2(acc[2], acc[3])};
      *reinterpret_cast<u32x2*>(a.out + out_row * kRowBytes + piece * 8) = v;
      if (piece == 0) a.lse[out_row] = lse;
    }
  }
  if (chunk && combined_here<G, kFlat>(it, m))
    arrive<T, G, kFlat, kRB>(a, it, hk, rs_o, rs_lse, m, words, s_last, *reinterpret_cast<MergeList*>(lds));
}

// Kinds of the kernel (kMode): plain; for batches with many short q tiles (decode steps); for batches whose q tiles
// may be narrow.
constexpr int kPlain = 0, kGated = 1, kNarrowTiles = 2;

// Pipeline of one workgroup.  A KV tile (64 keys, 4 pages) is the unit of the V staging
// and of the workgroup barrier; a half tile (32 keys, 2 pages) is the unit of the K staging and
// of the softmax pipeline.  Half tile h lives in slot h % 4 of a ring of four K buffers, V
// tile j in V buffer j % 2.
//   tile j        issues the global->LDS copies of V(j+1) and of K halves 2j+3, 2j+4
//                 (asynchronous, no VGPRs), runs half steps 2j and 2j+1, waits for the copies
//   half step h   phase 1: S(h+1) = K(h+1) Q^T on the MFMA pipe, exponentials of S(h) on the VALU
//                 phase 2: O^T += V(h)^T P(h)^T on the MFMA pipe, row max of S(h+1) on the VALU
//                 O is rescaled only if a row max moved far
// The two score register sets swap roles every half step, so a tile starts and ends with the
// same set and nothing is copied.  Each step of a phase is one MFMA, at most one LDS fragment
// fetch (4 MFMAs ahead of its use) and a slice of the VALU work; the order is pinned.
// kGated: wavefronts none of whose rows exists skip the arithmetic.  Worth it for batches with
// many short q tiles (decode steps); the plain variant is ~2 % faster when all tiles are full.
// kNarrowTiles, where the plan is of whole tiles: as kGated (16 sequences of 40 new tokens over 3000, 8 / 8 heads, 56.6
// us a layer without, 55.3 with; one of 256 over 1500, 32 / 8, 27.1, 27.2).
// kCB: blocks of 32 rows per wavefront.  1: q tiles of 128 rows, two workgroups per compute
// unit.  2: q tiles of 256 rows, one workgroup per compute unit with twice the registers: every
// K and V fragment read from LDS feeds two MFMAs, every tile copied to LDS serves twice the rows.
template <typename T, int G, int kMode, int kCB>
__global__ __launch_bounds__(kThreads, kCB == 1 ? 2 : 1) void attn_kernel(AttnArgs a) {
  constexpr bool kGate = kMode != kPlain, kNarrow = kMode == kNarrowTiles;
  constexpr int kWaveRows = 32 * kCB;       // rows per wavefront
  constexpr int TOK = kBM * kCB / G;        // tokens per q tile
  constexpr int kHalf = kBN / 2;
  constexpr int kHalfBytes = kTileBytes / 2;
  typedef typename Mfma<T>::vec8 vec8;
  // 4 K half tiles then 2 V tiles; reused as the output staging area at the end
  __shared__ __attribute__((aligned(1024))) char lds[4 * kTileBytes];
  __shared__ int s_redo;   // a row of the fixed-reference pass overflowed: run the pass again
  __shared__ int s_last;   // chunks' arrivals this workgroup was the last of
  __shared__ int s_second; // the neighbouring chunk's rows are there

  // (the division goes through the vector unit, and the compiler may leave its result there, and with
  // it the addresses that the copies below take from scalar registers; the builtin for this is dropped
  // on a value that is the same in all lanes; the s_nop is the wait state that reading a lane of a
  // register needs after a vector instruction wrote it, which the compiler does not add for assembly)
  int wi;
  asm("s_nop 1\n\tv_readfirstlane_b32 %0, %1" : "=s"(wi) : "v"(blockIdx.x / a.hkv));
  const int hk = blockIdx.x - wi * a.hkv;
  // The item record is requested together with the plan's header (the grid never exceeds the
  // room for records, whatever the header says): one memory round trip, with every argument the
  // look-ups behind it need already in registers.  (Left alone the compiler reads the header field
  // by field, a wait and a branch each, then the record, then the arguments.)
  const auto* rec = (const __attribute__((address_space(4))) i32x8*)(a.items + wi);
  i32x8 item = rec[0], item_b = rec[1];
  i32x8 hdr = *(const __attribute__((address_space(4))) i32x8*)a.hdr;
  int behind = a.behind;
  asm volatile("" : "+s"(behind));
  asm volatile("" ::"s"(a.pool_layer), "s"(a.begin), "s"(a.q), "s"(a.num_pages), "s"(a.total_q));
  asm volatile("" : "+s"(item), "+s"(item_b), "+s"(hdr));
  // the work list must come from a plan made for this very batch
  const bool narrow = kNarrow && (hdr[3] == kNarrowRows / G || hdr[3] == kNarrowRows / 2 / G);
  const bool ours = (hdr[0] == kPlanMagic) & (hdr[1] == head_counts(a.hkv, G)) & (wi < hdr[2]) &
                    (narrow | (hdr[3] == TOK)) & (hdr[4] == a.batch) & (hdr[5] == a.total_q);
  if (!ours) return;

  const int tid = threadIdx.x, lane = tid & 63;
  if (tid == 0) s_redo = s_last = 0;   // published by the barriers below
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, half = lane >> 5;

  const int seq = item[0], row0 = item[1];
  const int t0 = (item[2] & 0xffffff) << 1;          // first KV tile of the item (even)
  const int t1 = item[3] & 0x3ffffff;                // the one after its last
  const int chunk = item[4];                         // >= 0: one of several chunks
  const bool group = (item[3] & kItemGroup) != 0;    // shared-prefix item
  const int q_first = item[5];                       // the tile's first token in the q array
  const int ntok = (int)((uint32_t)item[2] >> 24) + 1;   // valid tokens in this tile (>= 1)
  const int table_off = item[6];
  const int pidx_cap = 4 * (t1 - 1) + (int)((uint32_t)item[3] >> 26 & 3);
  const int merge = item[7];                         // merge record, if chunk >= 0
  // a record that cannot come from the planner (a workspace written over by something else)
  const bool odd = ((unsigned)seq >= (unsigned)a.batch) | (row0 < 0) | (t1 <= t0) | (ntok > (narrow ? hdr[3] : TOK)) |
                   (q_first < 0) | ((int64_t)q_first + ntok > a.total_q) | (table_off < 0) |
                   ((chunk >= 0) & ((unsigned)merge >= (unsigned)hdr[6])) |
                   (group & (chunk < 0)) | ((kCB != 1) & (chunk >= 0));   // (ranges of wide q tiles are never cut)
  if (odd) return;
  // begin is read here, not taken from the plan (one plan may serve many decode steps)
  const int b = ((const_i32_ptr)a.begin)[seq];
  const Item it = {t0, t1, chunk, q_first, ntok, table_off, pidx_cap, merge, hdr[6], behind, group};
  if (kMode == kGated && ntok * G <= kFlatRows) {
    __shared__ float s_stat[2 * 4 * kFlatRows];   // maximum and sum per wavefront and row
    few_rows_item<T, G, 1, false>(a, it, hk, b, row0, item_b, lds, s_stat, s_last, false);
    return;
  }
  // (a prefix's items are few: with 32 rows they go that way beside whole tiles, too.  8 forks of 1024 tokens beside 100 new
  // ones, 32 / 8 heads, 23.0 us a layer, so 20.8.)
  if (kNarrow && (narrow | (ntok * G <= (group ? kNarrowRows : kFlatRows)))) {
    __shared__ float s_stat[2 * 4 * kNarrowRows];
    if (ntok * G <= kFlatRows) few_rows_item<T, G, 1, true>(a, it, hk, b, row0, item_b, lds, s_stat, s_last,
                                                                 narrow | (hdr[2] * a.hkv <= a.units));
    else few_rows_item<T, G, 2, true>(a, it, hk, b, row0, item_b, lds, s_stat, s_last, true);
    return;
  }

  // ---- global -> LDS copies (no VGPR staging) -------------------------------------
  // A wavefront's copy instruction fills 1 KiB of LDS linearly (lane L -> bytes 16 L..),
  // i.e. 4 rows.  A page is 16 rows: wave w fills rows 4 w + L/16 of the page (slots
  // 4 w..4 w+3); lane L fetches the 16-byte chunk that the swizzle wants at position L%16 of
  // that row.  Rows of keys at or beyond kv_len receive whatever the page holds (K: discarded
  // by the mask; V: zeroed in LDS before the last tile's P.V, since 0 x NaN would poison the
  // accumulators).
  const int ld_slot = 4 * wave + (lane >> 4), ld_pos = lane & 15;
  const char* pool_k = a.pool_layer + (int64_t)hk * kHeadPageBytes;
  const uint32_t k_lane_off = ld_slot * kRowBytes + ((ld_pos ^ ld_slot) << 4);
  const uint32_t v_lane_off = ld_slot * kRowBytes + ((ld_pos ^ ((ld_slot & 3) << 2)) << 4) +
                              (uint32_t)a.hkv * kHeadPageBytes;   // V run sits hkv blocks after K
  const uint32_t page_blocks = 2u * a.hkv;     // 4 KiB blocks per page
  const uint32_t lds_k = lds_addr(lds), lds_v = lds_k + 2 * kTileBytes;
  // wave-uniform address of this kv head's K run in the page of table entry pidx; entries
  // past the last needed one are replaced by the last needed one
  auto page_base = [&](int32_t pg) __attribute__((always_inline)) {
    pg = min(max(pg, 0), a.num_pages - 1);         // checked by the plan; stay in bounds anyway
    return pool_k + ((uint64_t)((uint32_t)pg * page_blocks) << 12);
  };
  auto copy_page = [&](const char* base, bool is_v, uint32_t lds_page) __attribute__((always_inline)) {   // 16 rows = 4 KiB
    copy16_to_lds(base, is_v ? v_lane_off : k_lane_off, lds_page + wave * 1024);
  };
  // The first tiles' copies - K halves 0, 1, 2 and V(0) of the item - need the record alone (it holds
  // the ids of table entries 4 t0 .. 4 t0 + 7): they leave before anything that depends on `begin`.
  // With the look-ups at the kernel's start in one request, one decode row over 1000 keys (32 / 8
  // heads): append, attention and merge of a layer 12.0 -> 11.4 us from first to last instruction;
  // eight rows (64 / 8 heads, 1024..4096 keys) 29.6 -> 29.0 us a layer.
  auto first_copies = [&]() __attribute__((always_inline)) {
    const char* pb[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) pb[i] = page_base(item_b[i]);
#pragma unroll
    for (int i = 0; i < 6; ++i) copy_page(pb[i], false, lds_k + i * 4096);
#pragma unroll
    for (int i = 0; i < 4; ++i) copy_page(pb[i], true, lds_v + i * 4096);
  };
  first_copies();
  // The position of the tile's first token.  The rows of a shared-prefix item are new tokens of
  // consecutive sequences; all of them lie beyond the prefix, so any position at or past the
  // item's last key serves.
  const int first_pos = group ? t1 * kBN : b + row0;
  // keys [64 t0, kv_len) are this item's: up to the end of its chunk, or of the tile's range
  const int kv_len = min(first_pos + ntok, t1 * kBN);
  const int n_kv_tiles = (kv_len + kBN - 1) / kBN;   // (absolute) index after the last KV tile
  const int n_halves = (kv_len + kHalf - 1) / kHalf;
  // half h is fully visible to every row of the q tile iff 32 (h+1) <= first_pos + 1
  const int n_full = (first_pos + 1) / kHalf;
  // A begin that no longer fits the item - negative, or so small that the item's first tile
  // lies past the range - skips the item before the page table is read (a chunk still arrives, with no
  // key in its rows); table indices never pass the last entry the plan validated for the sequence.
  const bool fits = b >= 0 && kv_len > kBN * t0;
  if (!fits) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the copies write this workgroup's LDS
    if (chunk < 0) return;
  }
  const int last_pidx = min((kv_len - 1) / kPage, pidx_cap);   // last entry that holds a needed key

  // this lane's query rows, one per row block
  int g[kCB], tt[kCB], my_pos[kCB];
  bool row_ok[kCB];
  // Q as the B operand: lane holds d = 16 kk + 8 half + [0,8) of its row, kk = 0..7
  vec8 qreg[kCB][8];
#pragma unroll
  for (int cb = 0; cb < kCB; ++cb) {
    const int r = wave * kWaveRows + cb * 32 + l32;    // row in tile
    g[cb] = r % G;                                     // token-major: the rows of a short tile
    tt[cb] = r / G;                                    // (a decode step's G rows) fill whole waves
    row_ok[cb] = tt[cb] < ntok;
    my_pos[cb] = first_pos + (row_ok[cb] ? tt[cb] : ntok - 1);   // causal limit of the row
    // (a row that does not exist reads the last one's q: no load under a condition; its results are
    // never stored)
    const int64_t q_row =
        ((int64_t)(q_first + min(tt[cb], ntok - 1)) * a.hq + hk * G + g[cb]) * kRowBytes;
#pragma unroll
    for (int kk = 0; kk < 8; ++kk)
      qreg[cb][kk] = __builtin_bit_cast(
          vec8, *reinterpret_cast<const u32x4*>(a.q + q_row + kk * 32 + half * 16));
  }
  // a wavefront none of whose rows exists only helps with the copies and the barriers
  const bool wave_active = !kGate || wave * kWaveRows < ntok * G;

  // ---- the page ids of the next copies -----------------------------------------------
  // The page ids of a tile's copies are fetched one tile early by a vector load (lane i & 7
  // holds table entry first + i).  It is an ordinary load, which the compiler tracks: wherever
  // the value is next needed (or moved, or spilled) the compiler waits for it, and since memory
  // operations complete in the order of their issue that wait also covers the copies issued
  // before it, which the compiler does not know of.  (As an untracked assembly load the register
  // could be spilled, under register pressure, before its data had arrived.)  arrive() is the
  // explicit wait for the copies - assembly statements, uncounted by the compiler - ahead of
  // the workgroup barrier.
  const int32_t* table_g = a.page_table + table_off;
  struct PageIds {
    int32_t reg;
    const int32_t* table;
    int lane7, last;
    __device__ __forceinline__ void issue(int first) {
      reg = __builtin_nontemporal_load(table + min(first + lane7, last));
    }
    __device__ __forceinline__ void arrive() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
    __device__ __forceinline__ int32_t value() const { return reg; }
  } ids;                                  // table entries of the next tile's copies
  ids.table = table_g;
  ids.lane7 = lane & 7;
  ids.last = last_pidx;
  auto wait_copies_and_sync = [&]() __attribute__((always_inline)) {
    ids.arrive();
    __syncthreads();
  };

  // ---- LDS fragment fetches ----------------------------------------------------------
  // K fragment f (0..7) of a half tile = d-step kk: rows l32, 16-byte chunk 2 kk + half.
  // V fragment g (0..7) of a half tile (rows crow..crow+31 of its tile): 16-key step st = g >> 2,
  // d chunk dc = g & 3; a 16-lane group reads 4 keys x 16 d, lane j supplies key (j/4) and d-quad
  // (j%4); the two reads cover accumulator registers 8 st..8 st+7, i.e. for this lane-half the
  // keys 16 st + {0..3} + 4 half and 16 st + 8 + {0..3} + 4 half.
  const int j16 = lane & 15, gq = (lane >> 4) & 1;
  auto k_frag = [&](uint32_t khalf, int f) __attribute__((always_inline)) {
    return *reinterpret_cast<const vec8 __attribute__((address_space(3)))*>(
        (size_t)(khalf + k_swz(l32, 2 * f + half)));
  };
  auto v_frag = [&](uint32_t vtile, int crow, int gi) __attribute__((always_inline)) {
    const int st = gi >> 2, dc = gi & 3;
    const int key_lo = crow + st * 16 + 4 * half + (j16 >> 2);
    const int chunk = dc * 4 + gq * 2 + ((j16 & 3) >> 1);
    const int sub = (j16 & 1) * 8;
    s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (lds_s16x4_ptr)(size_t)(vtile + v_swz(key_lo, chunk) + sub));
    s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (lds_s16x4_ptr)(size_t)(vtile + v_swz(key_lo + 8, chunk) + sub));
    return __builtin_bit_cast(vec8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };

  // key held by accumulator register i of half h: 32 h + 8 (i/4) + 4 half + i%4
  auto mask_half = [&](int h, f32x16& sc, int cb) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int key = h * kHalf + 8 * (i >> 2) + 4 * half + (i & 3);
      if (key > my_pos[cb]) sc[i] = -INFINITY;
    }
  };
  // the other 16 keys of the row's half tile sit in lane l ^ 32: swap the wave's halves on the VALU
  // with one v_permlane32_swap: given the value in both operands, the first comes back holding
  // the lower half's value in both halves and the second the upper half's.  Written as assembly
  // (with the two wait states the instruction needs after a vector write of its operands):
  // through __builtin_amdgcn_permlane32_swap this compiler hands out the first result twice.
  auto max_across_halves = [&](float mx) __attribute__((always_inline)) {
    uint32_t lo = __builtin_bit_cast(uint32_t, mx), hi = lo;
    asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(lo), "+v"(hi));
    return fmaxf(__builtin_bit_cast(float, lo), __builtin_bit_cast(float, hi));
  };

  f32x16 o_acc[kCB][4];
  float m_run[kCB], l_run[kCB];           // reference score of the row (raw), this lane's partial sum
  float mx_cur[kCB];                      // row max of the half tile about to be exponentiated
  const float c2 = a.scale_log2;
  const f32x16 zero16 = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  constexpr int kAhead = 4;               // fragments in flight
  vec8 kf[kAhead];                        // first K fragments of the next phase 1
  f32x16 s_a[kCB], s_b[kCB];

  // ---- one half step.  s_cur = S(h) in, s_next = S(h+1) out (computed even when half h+1
  //      does not exist: its LDS rows are then stale, the result is never used).
  //      k_next: LDS address of K half h+1; k_after: of K half h+2, whose first fragments are
  //      fetched at the end of this step if fetch_after; v_cur/crow: V tile and row offset of
  //      half h.  mask_next: half h+1 reaches the causal diagonal.
  //      fixed_ref: the row's reference score stays where the prologue put it (see run_pass):
  //      no row max, no rescale, and the exponentials of the last kPairsLate register pairs move
  //      into phase 2, whose VALU slots the row max no longer needs.
  auto half_step = [&](auto fixed_ref, int h, uint32_t k_next, bool fetch_after, uint32_t k_after,
                       uint32_t v_cur, int crow, f32x16 (&s_cur)[kCB], f32x16 (&s_next)[kCB],
                       bool mask_next, auto&& slot_extra) __attribute__((always_inline)) {
    constexpr bool kFixed = decltype(fixed_ref)::value;
    constexpr int kPairs = 8 * kCB;                       // register pairs of S(h), all row blocks
    constexpr int kLate = kFixed ? kPairsLate * kCB : 0;  // ... of which phase 2 takes this many
    vec8 vf[kAhead];
    if constexpr (!kFixed) {
      // ---- move the reference max (and rescale O, l) only when some row's max rose by more
      //      than 2^8 in the exp2 domain: p stays below 2^8, sums stay exact
      bool moved = false;
#pragma unroll
      for (int cb = 0; cb < kCB; ++cb) moved |= (mx_cur[cb] - m_run[cb]) * c2 > 8.f;
      if (__builtin_amdgcn_ballot_w64(moved) != 0) {
#pragma unroll
        for (int cb = 0; cb < kCB; ++cb) {
          const float m_new = fmaxf(m_run[cb], mx_cur[cb]);
          const float alpha = __builtin_amdgcn_exp2f((m_run[cb] - m_new) * c2);
          m_run[cb] = m_new;
          l_run[cb] *= alpha;
#pragma unroll
          for (int dc = 0; dc < 4; ++dc)
#pragma unroll
            for (int i = 0; i < 16; ++i) o_acc[cb][dc][i] *= alpha;
        }
      }
    }
    float mc2[kCB];
#pragma unroll
    for (int cb = 0; cb < kCB; ++cb) mc2[cb] = m_run[cb] * c2;
    uint32_t p_pk[kCB][8];
    // softmax of register pair t of S(h) of row block cb (registers 2t, 2t+1 -> packed operand
    // word t).  The row sum takes the unrounded values: LSE must not inherit P's 2-byte rounding.
    // (The empty assembly statement keeps the additions here, beside their exponentials: left
    // alone the compiler gathers them at the end of the half step and keeps all values live.)
    auto soft_pair = [&](int cb, int t) __attribute__((always_inline)) {
      const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s_cur[cb][2 * t], c2, -mc2[cb]));
      const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s_cur[cb][2 * t + 1], c2, -mc2[cb]));
      l_run[cb] += p0 + p1;
      asm volatile("" : "+v"(l_run[cb]));
      p_pk[cb][t] = Mfma<T>::pack2(p0, p1);
    };
    // pairs in the order phase 2 needs them: words 0..3 of every row block, then words 4..7
    auto soft_nth = [&](int i) __attribute__((always_inline)) {
      soft_pair((i / 4) % kCB, (i / (4 * kCB)) * 4 + i % 4);
    };
    __builtin_amdgcn_sched_barrier(0);
    // ---- phase 1: 8 steps.  Step t: d-step t of S(h+1) for every row block (one K fragment
    //      feeds kCB MFMAs); beside each MFMA the softmax of a register pair of S(h).
#pragma unroll
    for (int t = 0; t < 8; ++t) {
#pragma unroll
      for (int cb = 0; cb < kCB; ++cb) {
        if (t * kCB + cb < kPairs - kLate) soft_nth(t * kCB + cb);
        if constexpr (kFixed && kCB == 2) {
          // (nothing reads these registers before the next half step's softmax, a whole phase
          // of MFMAs later, except the mask below, which waits for the matrix pipe first)
          if (t == 0) Mfma<T>::run_v0(kf[t % kAhead], qreg[cb][t], s_next[cb]);
          else Mfma<T>::run_v(kf[t % kAhead], qreg[cb][t], s_next[cb]);
        } else {
          s_next[cb] = Mfma<T>::run(kf[t % kAhead], qreg[cb][t], t == 0 ? zero16 : s_next[cb]);
        }
        if (cb + 1 < kCB) __builtin_amdgcn_sched_barrier(0);
      }
      if (t + kAhead < 8) kf[t % kAhead] = k_frag(k_next, t + kAhead);
      else vf[t % kAhead] = v_frag(v_cur, crow, t + kAhead - 8);
      slot_extra(t);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (mask_next) {
      // the scores may come from MFMAs the compiler does not see as such: let the last of them
      // (8 passes of 4 cycles) leave the pipe before vector instructions rewrite its registers
      if constexpr (kFixed && kCB == 2) asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 7" ::: "memory");
#pragma unroll
      for (int cb = 0; cb < kCB; ++cb) mask_half(h + 1, s_next[cb], cb);
    }
    // ---- phase 2: 8 steps.  Step u: V fragment u (16-key step st = u >> 2 -> operand words
    //      4 st..4 st+3, d chunk dc = u & 3) for every row block; beside the MFMAs the row max
    //      over register pair u of S(h+1), or the softmax pairs phase 1 left over.
    float mx[kCB];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int st = u >> 2, dc = u & 3;
#pragma unroll
      for (int cb = 0; cb < kCB; ++cb) {
        u32x4 pw = {p_pk[cb][4 * st], p_pk[cb][4 * st + 1], p_pk[cb][4 * st + 2], p_pk[cb][4 * st + 3]};
        o_acc[cb][dc] = Mfma<T>::run(vf[u % kAhead], __builtin_bit_cast(vec8, pw), o_acc[cb][dc]);
        if constexpr (kFixed) {
          if (u * kCB + cb < kLate) soft_nth(kPairs - kLate + u * kCB + cb);   // words 4..7: first read at step 4
        } else {
          mx[cb] = u == 0 ? fmaxf(s_next[cb][0], s_next[cb][1])
                          : max3(mx[cb], s_next[cb][2 * u], s_next[cb][2 * u + 1]);
        }
        if (cb + 1 < kCB) __builtin_amdgcn_sched_barrier(0);
      }
      if (u + kAhead < 8) vf[u % kAhead] = v_frag(v_cur, crow, u + kAhead);
      else if (fetch_after) kf[u % kAhead] = k_frag(k_after, u + kAhead - 8);
      slot_extra(8 + u);
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (!kFixed) {
#pragma unroll
      for (int cb = 0; cb < kCB; ++cb) mx_cur[cb] = max_across_halves(mx[cb]);
    }
  };

  // ---- the copies of one tile.  par = j & 1 fixes every LDS address of the tile: K halves 2j+1,
  //      2j+2 are read from ring slots 1, 2 (even j) or 3, 0 (odd j) while halves 2j+3, 2j+4 are
  //      copied into the other two; V(j) is read from V buffer par while V(j+1) is copied into
  //      the other.  Table entries 4j+4 .. 4j+9 are involved: V(j+1) is entries +4..+7, K halves
  //      2j+3, 2j+4 are +6..+9.  Every lane turns the id it holds into its page's address (two
  //      vector instructions); the six addresses then move to scalar registers.
  const uint64_t pool_k_u = (uint64_t)(size_t)pool_k;
  const uint32_t page_stride_b = page_blocks << 12;
  struct TilePages { const char* pb[6]; };
  auto tile_pages = [&](int jt) __attribute__((always_inline)) {
    const int32_t pg = min(max(ids.value(), 0), a.num_pages - 1);   // checked by the plan; stay in bounds anyway
    const uint64_t addr = pool_k_u + (uint64_t)(uint32_t)pg * page_stride_b;
    const uint32_t lo = (uint32_t)addr, hi = (uint32_t)(addr >> 32);
    TilePages tp;
#pragma unroll
    for (int i = 0; i < 6; ++i)
      tp.pb[i] = (const char*)(size_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane(hi, i) << 32) |
                                       (uint32_t)__builtin_amdgcn_readlane(lo, i));
    ids.issue(4 * jt + 8);
    return tp;
  };
  // copy c of the tile's eight: the pages of K half 2j+3, the first two of V(j+1), K half 2j+4,
  // the last two of V(j+1) - the order in which the next tile needs them
  auto tile_copy = [&](const TilePages& tp, const int par, int c) __attribute__((always_inline)) {
    const uint32_t k_h3 = lds_k + (par ? 1 : 3) * kHalfBytes;     // K half 2j+3 (copy target)
    const uint32_t k_h4 = lds_k + (par ? 2 : 0) * kHalfBytes;     // K half 2j+4 (copy target)
    const uint32_t v_nxt = lds_v + (par ^ 1) * kTileBytes;
    switch (c) {
      case 0: copy_page(tp.pb[2], false, k_h3); break;
      case 1: copy_page(tp.pb[3], false, k_h3 + 4096); break;
      case 2: copy_page(tp.pb[0], true, v_nxt); break;
      case 3: copy_page(tp.pb[1], true, v_nxt + 4096); break;
      case 4: copy_page(tp.pb[4], false, k_h4); break;
      case 5: copy_page(tp.pb[5], false, k_h4 + 4096); break;
      case 6: copy_page(tp.pb[2], true, v_nxt + 2 * 4096); break;
      default: copy_page(tp.pb[3], true, v_nxt + 3 * 4096); break;
    }
  };
  // last tile: zero the V rows of keys >= kv_len (their P is 0, their bytes are arbitrary)
  auto zero_v_tail = [&](int jt, const int par) __attribute__((always_inline)) {
    const uint32_t v_cur = lds_v + par * kTileBytes;
    const int valid = kv_len - jt * kBN;
    const u32x4 zero = {0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = i * 16 + (tid >> 4);
      if (row >= valid)
        *reinterpret_cast<u32x4 __attribute__((address_space(3)))*>(
            (size_t)(v_cur + row * kRowBytes + (tid & 15) * 16)) = zero;
    }
    __syncthreads();
  };
  auto tile_copies = [&](int jt, const int par, bool in_main_loop) __attribute__((always_inline)) {
    if (in_main_loop || jt + 1 < n_kv_tiles) {
      const TilePages tp = tile_pages(jt);
#pragma unroll
      for (int c = 0; c < 8; ++c) tile_copy(tp, par, c);
    } else if (kv_len < (jt + 1) * kBN) {
      zero_v_tail(jt, par);
    }
  };

  // ---- one pass over the item's KV range, from its first tile: leaves o_acc, m_run, l_run.
  //      fixed_ref = false: the row's reference score follows the running row max (moved, with
  //      a rescale of O and l, when a half tile's max exceeds it by more than 2^8 in the exp2
  //      domain), so p <= 2^8 whatever the scores are.
  //      fixed_ref = true: the reference stays at the row max of the first half tile.  Any
  //      reference gives the same O and LSE as long as nothing overflows; this one costs no row
  //      max, no exchange between the wavefront's halves and no branch per half step.  Its p is
  //      unbounded, so it is only used where P keeps fp32's exponent range (bf16), and the
  //      caller checks the row sums afterwards.
  auto run_pass = [&](auto fixed_ref) __attribute__((always_inline)) {
#pragma unroll
    for (int cb = 0; cb < kCB; ++cb) {
#pragma unroll
      for (int dc = 0; dc < 4; ++dc)
#pragma unroll
        for (int i = 0; i < 16; ++i) o_acc[cb][dc][i] = 0.f;
      m_run[cb] = -INFINITY;
      l_run[cb] = 0.f;
    }
    // ---- prologue: K halves 0, 1, 2 and V(0) are in flight (first_copies); S(half 0) ---------
    ids.issue(4 * t0 + 4);
    wait_copies_and_sync();
    if (wave_active) {
#pragma unroll
      for (int f = 0; f < 8; ++f) {
        const vec8 kfr = k_frag(lds_k, f);
#pragma unroll
        for (int cb = 0; cb < kCB; ++cb) {
          if constexpr (decltype(fixed_ref)::value && kCB == 2) {
            if (f == 0) Mfma<T>::run_v0(kfr, qreg[cb][f], s_a[cb]);
            else Mfma<T>::run_v(kfr, qreg[cb][f], s_a[cb]);
          } else {
            s_a[cb] = Mfma<T>::run(kfr, qreg[cb][f], f == 0 ? zero16 : s_a[cb]);
          }
        }
      }
      // (MFMAs written as assembly: the matrix pipe must have drained before their results are read)
      if constexpr (decltype(fixed_ref)::value && kCB == 2)
        asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 7" ::: "memory");
#pragma unroll
      for (int cb = 0; cb < kCB; ++cb) {
        if (n_full <= 2 * t0) mask_half(2 * t0, s_a[cb], cb);
        float mx = fmaxf(s_a[cb][0], s_a[cb][1]);
#pragma unroll
        for (int i = 2; i < 16; i += 2) mx = max3(mx, s_a[cb][i], s_a[cb][i + 1]);
        mx_cur[cb] = max_across_halves(mx);
        if constexpr (decltype(fixed_ref)::value) m_run[cb] = mx_cur[cb];
      }
    }
    __syncthreads();   // every wave has read K half 0 before tile 0 overwrites its slot

    // A wavefront none of whose rows exists (short tiles: a decode step has G rows) takes its
    // share of the copies and of the barriers, tile by tile, and nothing else.
    if (kGate && !wave_active) {
      for (int jt = t0; jt < n_kv_tiles; ++jt) {
        tile_copies(jt, jt & 1, false);
        wait_copies_and_sync();
      }
      return;
    }

    // ---- one tile
    auto tile = [&](int jt, const int par, bool mask0, bool mask1,
                    bool in_main_loop) __attribute__((always_inline)) {
      const uint32_t k_h1 = lds_k + (par ? 3 : 1) * kHalfBytes;     // K half 2j+1
      const uint32_t k_h2 = lds_k + (par ? 0 : 2) * kHalfBytes;     // K half 2j+2
      const uint32_t v_cur = lds_v + par * kTileBytes;
#pragma unroll
      for (int f = 0; f < kAhead; ++f) kf[f] = k_frag(k_h1, f);
      auto nothing = [](int) __attribute__((always_inline)) {};
      if (in_main_loop) {
        // the tile's copies go out one per MFMA slot of the first half step's second phase
        // (addresses in the slot before), under the matrix pipe's work instead of ahead of it
        TilePages tp;
        half_step(fixed_ref, 2 * jt, k_h1, true, k_h2, v_cur, 0, s_a, s_b, mask0,
                  [&](int slot) __attribute__((always_inline)) {
                    if (slot == kCopySlot0 - 1) tp = tile_pages(jt);
                    if (slot >= kCopySlot0 && slot < kCopySlot0 + 8) tile_copy(tp, par, slot - kCopySlot0);
                  });
      } else {
        tile_copies(jt, par, false);
        half_step(fixed_ref, 2 * jt, k_h1, true, k_h2, v_cur, 0, s_a, s_b, mask0, nothing);
      }
      if (in_main_loop || 2 * jt + 1 < n_halves)
        half_step(fixed_ref, 2 * jt + 1, k_h2, false, 0, v_cur, kHalf, s_b, s_a, mask1, nothing);
      wait_copies_and_sync();
    };

    // Tiles whose two half steps need no mask on their successor halves (2j+1, 2j+2 below the
    // diagonal) run two per iteration with constant LDS addresses; the rest follow one by one.
    const int n_main = max(t0, min(n_full - 2, 2 * n_kv_tiles - 2) / 2);   // tiles j with 2j+2 < n_full
    int jt = t0;
    for (; jt + 1 < n_main; jt += 2) {
      tile(jt, 0, false, false, true);
      tile(jt + 1, 1, false, false, true);
    }
    for (; jt < n_kv_tiles; ++jt)
      tile(jt, jt & 1, 2 * jt + 1 >= n_full, 2 * jt + 2 >= n_full, false);
  };

  if (fits) {
    if constexpr (kTryFixedRef<T>) {
      // First with the fixed reference.  A row whose sum left the range in which nothing can have
      // overflowed (or is not a number) sends the whole workgroup through the pass again with the
      // moving reference; on scores like the workloads' (a few units wide) that never happens.
      run_pass(std::true_type{});
      bool sums_ok = true;
      float o_chk = 0.f;                     // NaN if any accumulator is infinite or not a number
#pragma unroll
      for (int cb = 0; cb < kCB; ++cb) {
        sums_ok = sums_ok && l_run[cb] + __shfl_xor(l_run[cb], 32) < kFixedRefSumLimit;
#pragma unroll
        for (int dc = 0; dc < 4; ++dc)
#pragma unroll
          for (int i = 0; i < 16; ++i) o_chk = __builtin_fmaf(o_acc[cb][dc][i], 0.f, o_chk);
      }
      const bool bad = wave_active && !(sums_ok && o_chk == 0.f);
      if (__builtin_amdgcn_ballot_w64(bad) != 0 && lane == 0) s_redo = 1;
      __syncthreads();
      if (s_redo != 0) {
        first_copies();
        run_pass(std::false_type{});
      }
    } else {
      run_pass(std::false_type{});
    }
  }

  // ---- epilogue: normalise ----
  bool row_live[kCB];                     // the row exists and this wavefront has it
  float lse_row[kCB];
#pragma unroll
  for (int cb = 0; cb < kCB; ++cb) {
    row_live[cb] = row_ok[cb] && wave_active;
    if (fits) {
      const float l_tot = l_run[cb] + __shfl_xor(l_run[cb], 32), inv = 1.f / l_tot;
      lse_row[cb] = m_run[cb] * a.scale + __logf(l_tot);
#pragma unroll
      for (int dc = 0; dc < 4; ++dc)
#pragma unroll
        for (int i = 0; i < 16; ++i) o_acc[cb][dc][i] *= inv;
    } else {
      lse_row[cb] = -INFINITY;
#pragma unroll
      for (int dc = 0; dc < 4; ++dc) o_acc[cb][dc] = zero16;
    }
  }

  if (kCB == 1 && chunk >= 0) {
    // ---- one of several chunks (see MergeRec).  Partial rows reach the memory all XCDs see before
    //      the workgroup says so, and are read after the word that says so.  Nobody waits for anybody.
    //      As a launch of its own behind this one, reading every partial row, the merge took 3.6 us of the
    //      12 us a layer of one decode row over 1000 keys needs, 10 of the 63 us of 500 new tokens over
    //      4500 (four chunks of 128 rows), and 4.7 us where nothing was cut; now 2.5, 4.4 and none
    //      (32 / 8 heads; per layer 13.9 -> 12.9 and 70 -> 60 us).
    const buffer_rsrc rs_o = make_rsrc(a.part_o, (uint32_t)a.part_cap * a.hq * 512u);
    const buffer_rsrc rs_lse = make_rsrc(a.part_lse, (uint32_t)a.part_cap * a.hq * 4u);
    i32x8 m = *(const __attribute__((address_space(4))) i32x8*)(a.merges + merge);
    const int words = ((const_i32_ptr)a.hdr)[10];
    const int rows = ntok * G;
    const uint32_t step = ntok * a.hq;                        // partial rows of a chunk
    const uint32_t chunk0 = m[3] * a.hq + hk * rows;          // of chunk 0 (of a tile, not of a group)
    // A row's 32 pieces of 16 bytes lie row by row, for readers that take rows, or as the registers lie
    // (a store fills 1 KiB).  Registers 4 j .. 4 j + 3 of o_acc[dc] hold d = 32 dc + 8 j + 4 half +
    // {0..3}: piece 2 i + half with i = 4 dc + j.  Where piece `half` of row r is, if a chunk's rows
    // start at row0, and from one i to the next:
    struct Place { uint32_t byte, step; };
    auto by_row = [&](uint32_t row0, int r, int) __attribute__((always_inline)) {
      return Place{(row0 + r) * 512u + half * 16, 32u};
    };
    auto by_reg = [&](uint32_t row0, int r, int of_rows) __attribute__((always_inline)) {
      return Place{row0 * 512u + r * 32u + half * 16, of_rows * 32u};
    };
    auto tile_row = [&](int cb) __attribute__((always_inline)) { return wave * kWaveRows + cb * 32 + l32; };
    auto write_rows = [&](uint32_t row0, bool flat, auto scope) __attribute__((always_inline)) {
      constexpr int kScope = decltype(scope)::value;
#pragma unroll
      for (int cb = 0; cb < kCB; ++cb) {
        if (!row_live[cb]) continue;
        const Place at = flat ? by_row(row0, tile_row(cb), rows) : by_reg(row0, tile_row(cb), rows);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const f32x16& o = o_acc[cb][i >> 2];
          const int j = 4 * (i & 3);
          store_part<kScope>(rs_o, at.byte + i * at.step, f32x4{o[j], o[j + 1], o[j + 2], o[j + 3]});
        }
        if (half == 0) store_part<kScope>(rs_lse, (row0 + tile_row(cb)) * 4u, lse_row[cb]);
      }
    };
    constexpr std::integral_constant<int, kDeviceScope> in_launch{};
    auto read_row = [&](Place at, f32x4 (&o)[16]) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < 16; ++i) o[i] = load_part4<kDeviceScope>(rs_o, at.byte + i * at.step);
    };

    const bool tree = rows > kFlatRows && !group && !(behind & kTreesBehind);
    if (tree) {
      uint32_t* word0 = reinterpret_cast<uint32_t*>(a.part_lse) + (int64_t)a.part_cap * a.hq - 1 -
                        ((int64_t)merge * a.hkv + hk) * words - 1;
      int idx = chunk, count = m[2], node0 = 0;
      for (int level = 0; count > 1; ++level) {
        if ((idx ^ 1) < count) {
          const int node = node0 + (idx >> 1);
          uint32_t* word = word0 - (node >> 5);
          const uint32_t bit = 1u << (node & 31);
          if (tid == 0) {
            const bool there = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & bit;
            if (there) atomicXor(word, bit);
            s_second = there;
          }
          __syncthreads();
          bool second = s_second != 0;
          __syncthreads();
          if (!second) {
            write_rows(chunk0 + (idx << level) * step, false, in_launch);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            if (tid == 0) s_second = (atomicXor(word, bit) & bit) != 0;
            __syncthreads();
            second = s_second != 0;
            __syncthreads();
            if (!second) return;
          }
          const uint32_t other = chunk0 + ((idx ^ 1) << level) * step;
#pragma unroll
          for (int cb = 0; cb < kCB; ++cb) {
            if (!row_live[cb]) continue;
            const float lse = load_part<kDeviceScope>(rs_lse, (other + tile_row(cb)) * 4u);
            f32x4 o[16];
            read_row(by_reg(other, tile_row(cb), rows), o);
            if (lse == -INFINITY && lse_row[cb] == -INFINITY) continue;   // neither holds a key of this row
            const float mx = fmaxf(lse, lse_row[cb]);
            const float w0 = __expf(lse_row[cb] - mx), w1 = __expf(lse - mx), den = w0 + w1;
            const float f0 = w0 / den, f1 = w1 / den;
            lse_row[cb] = mx + __logf(den);
            // the same sum whichever of the two is the second: products, then their sum
#pragma unroll
            for (int i = 0; i < 16; ++i)
#pragma unroll
              for (int j = 0; j < 4; ++j) {
#pragma clang fp contract(off)
                const float x = o_acc[cb][i >> 2][4 * (i & 3) + j] * f0, y = o[i][j] * f1;
                o_acc[cb][i >> 2][4 * (i & 3) + j] = x + y;
              }
          }
        }
        node0 += (count + 1) >> 1;
        count = (count + 1) >> 1;
        idx >>= 1;
      }
    }
    if (!tree || m[4] > 0) {
      const uint32_t row0 = tree ? chunk0 : first_part_row<G>(a, it, hk, m);
      // (launches that may have narrow tiles never combine a prefix's chunks; 16 rows went another way above)
      if (kNarrow || !combined_here<G, kFlatRows>(it, m)) {
        write_rows(row0, !tree, std::integral_constant<int, kLaunchScope>{});
        return;
      }
      if constexpr (!kNarrow) {
        write_rows(row0, !tree, in_launch);
        arrive<T, G, kFlatRows, 1>(a, it, hk, rs_o, rs_lse, m, words, s_last, *reinterpret_cast<MergeList*>(lds));
        return;
      }
    }
  }
  if (kGate && !wave_active) return;
  if (kCB == 1 && chunk >= 0) {      // no chunk of these rows was computed: nothing is written
    bool some = false;
#pragma unroll
    for (int cb = 0; cb < kCB; ++cb) some |= row_live[cb] && lse_row[cb] != -INFINITY;
    if (__builtin_amdgcn_ballot_w64(some) == 0) return;
  }

  // ---- the tile's result: stage O through LDS for full-row stores, write LSE ----
  // 8 KiB per wave and row block; all tiles are consumed
#pragma unroll
  for (int cb = 0; cb < kCB; ++cb) {
    char* stage = lds + (wave * kCB + cb) * (32 * kRowBytes);
#pragma unroll
    for (int dc = 0; dc < 4; ++dc)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        // registers 4j..4j+3 hold d = 32 dc + 8 j + 4 half + {0..3}: 8 bytes of chunk 4 dc + j
        u32x2 w;
        w[0] = Mfma<T>::pack2(o_acc[cb][dc][4 * j], o_acc[cb][dc][4 * j + 1]);
        w[1] = Mfma<T>::pack2(o_acc[cb][dc][4 * j + 2], o_acc[cb][dc][4 * j + 3]);
        *reinterpret_cast<u32x2*>(stage + k_swz(l32, 4 * dc + j) + half * 8) = w;
      }
    if (row_live[cb] && half == 0)
      a.lse[(int64_t)(q_first + tt[cb]) * a.hq + hk * G + g[cb]] = lse_row[cb];
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int cb = 0; cb < kCB; ++cb) {
    const char* stage = lds + (wave * kCB + cb) * (32 * kRowBytes);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int lr = 4 * i + (lane >> 4);               // row of this block's 32
      const int rr = wave * kWaveRows + cb * 32 + lr, gg = rr % G, t2 = rr / G;
      const u32x4 v = *reinterpret_cast<const u32x4*>(stage + k_swz(lr, lane & 15));
      if (t2 < ntok)
        *reinterpret_cast<u32x4*>(a.out + ((int64_t)(q_first + t2) * a.hq + hk * G + gg) * kRowBytes +
                                  (lane & 15) * 16) = v;
    }
  }
}

// The chunks that attn_kernel's launch does not combine: a workgroup per merge record, 8 rows and kv head
// (`blocks` of them share a record's rows), or as many in turn.  It does nothing where the plan found no
// group or cut nothing, which takes the longer the more workgroups have to find that out.
template <typename T, int G>
__global__ __launch_bounds__(kThreads) void merge_kernel(AttnArgs a, int blocks) {
  const i32x8 hdr = *(const __attribute__((address_space(4))) i32x8*)a.hdr;
  const bool trees = !(a.behind & kTreesBehind);
  // (chunks of narrow q tiles are counted in the launch)
  const bool none = hdr[6] == 0 || (((const_i32_ptr)a.hdr)[8] == 0 && (trees || hdr[3] * G < kBM));
  if (hdr[0] != kPlanMagic || hdr[1] != head_counts(a.hkv, G) || none || hdr[4] != a.batch || hdr[5] != a.total_q) return;
  const buffer_rsrc rs_o = make_rsrc(a.part_o, (uint32_t)a.part_cap * a.hq * 512u);
  const buffer_rsrc rs_lse = make_rsrc(a.part_lse, (uint32_t)a.part_cap * a.hq * 4u);
  const int64_t per_rec = (int64_t)a.hkv * blocks;
  for (int64_t w = blockIdx.x; w < hdr[6] * per_rec; w += gridDim.x) {
    const int rec = __builtin_amdgcn_readfirstlane((int)(w / per_rec)), at = (int)(w - rec * per_rec);
    const i32x8 m = *(const __attribute__((address_space(4))) i32x8*)(a.merges + rec);
    if (!(m[4] > 0 ? a.behind & kGroupsBehind : !trees && m[1] * G > kFlatRows)) continue;
    const int block = __builtin_amdgcn_readfirstlane(at / a.hkv), hk = at - block * a.hkv;
    merge_rows<T, G, kLaunchScope, 1, kMergeAhead>(
        a, rs_o, rs_lse, hk, m[1], kFlatRows, trees, block, blocks,
        [&](int, int& first) __attribute__((always_inline)) { first = 0; return m; });
  }
}

template <typename T>
void launch_merge(int G, dim3 grid, int blocks, hipStream_t hs, const AttnArgs& a) {
  switch (G) {
    case 1: hipLaunchKernelGGL((merge_kernel<T, 1>), grid, dim3(kThreads), 0, hs, a, blocks); break;
    case 2: hipLaunchKernelGGL((merge_kernel<T, 2>), grid, dim3(kThreads), 0, hs, a, blocks); break;
    case 4: hipLaunchKernelGGL((merge_kernel<T, 4>), grid, dim3(kThreads), 0, hs, a, blocks); break;
    default: hipLaunchKernelGGL((merge_kernel<T, 8>), grid, dim3(kThreads), 0, hs, a, blocks); break;
  }
}

template <typename T, int kMode, int kCB>
mc_status launch_attn_g(int G, dim3 grid, hipStream_t hs, const AttnArgs& a) {
  switch (G) {
    case 1: hipLaunchKernelGGL((attn_kernel<T, 1, kMode, kCB>), grid, dim3(kThreads), 0, hs, a); break;
    case 2: hipLaunchKernelGGL((attn_kernel<T, 2, kMode, kCB>), grid, dim3(kThreads), 0, hs, a); break;
    case 4: hipLaunchKernelGGL((attn_kernel<T, 4, kMode, kCB>), grid, dim3(kThreads), 0, hs, a); break;
    case 8: hipLaunchKernelGGL((attn_kernel<T, 8, kMode, kCB>), grid, dim3(kThreads), 0, hs, a); break;
    default: return MC_ERR_UNSUPPORTED;
  }
  return mc::launch_status();
}

template <typename T>
mc_status launch_attn(int G, int mode, int row_blocks, dim3 grid, hipStream_t hs, const AttnArgs& a) {
  if (row_blocks == 2) return launch_attn_g<T, kPlain, 2>(G, grid, hs, a);
  switch (mode) {
    case kNarrowTiles: return launch_attn_g<T, kNarrowTiles, 1>(G, grid, hs, a);
    case kGated: return launch_attn_g<T, kGated, 1>(G, grid, hs, a);
    default: return launch_attn_g<T, kPlain, 1>(G, grid, hs, a);
  }
}

// Workgroups of the attention kernel the current GPU runs at a time: two per compute unit
// (one with the wide q tiles).
// The compute-unit count is asked for once per device (the query costs microseconds, which a
// decode step notices); the current device is a thread-local read.
int device_slots(int row_blocks = 1) {
  constexpr int kDevs = 64;
  static std::atomic<int> cached[kDevs];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0) return -1;
  if (dev < kDevs) {
    const int c = cached[dev].load(std::memory_order_relaxed);
    if (c > 0) return row_blocks == 2 ? c / 2 : c;
  }
  int cus = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      cus <= 0)
    return -1;
  if (dev < kDevs) cached[dev].store(2 * cus, std::memory_order_relaxed);
  return row_blocks == 2 ? cus : 2 * cus;
}

// The planner cuts KV ranges only if the q tiles times kv heads are fewer than kRoundsWanted per
// slot; the number of q tiles is at least total_q / tile_tokens, which the host knows.
bool may_cut(const WorkspaceLayout& w, int hkv, int slots) {
  return w.part_cap > 0 && (int64_t)(w.max_tiles - w.batch) * hkv < (int64_t)kRoundsWanted * slots;
}

// Whether the planner may take q tiles of fewer rows (narrow_rows): at most a workgroup of kNarrowRows rows a compute
// unit, few sequences, and more new tokens than those.  By the batch's sizes, because planner and attention kernel
// are others then: with these paths, which they never take, the others took 0.2 to 0.4 us longer a launch (one
// decode row, eight layers, 81.7 -> 84.1 us).  A batch that may have narrow tiles and keeps whole ones pays that (one
// range of 256 tokens over 1500, 32 / 8 heads, 26.3 -> 26.8 us a layer).
bool may_narrow(int32_t batch, int32_t total_q, int G, int hkv, int slots) {
  return batch <= kNarrowBatch && total_q > batch && (int64_t)total_q * G * hkv <= (int64_t)kNarrowRows * (slots / 2);
}

// Shared-prefix groups are made of sequences with one new token each: worth looking for only
// when the batch could hold a fair share of those (fewer than two q tiles' worth of new tokens
// per sequence on average), and possible only with room for partial rows.
bool may_group(const WorkspaceLayout& w, int32_t total_q, int tile_tokens) {
  return w.part_cap > 0 && w.batch >= 2 && w.batch <= kCuTilesInLds &&
         (int64_t)total_q < 2ll * w.batch * tile_tokens;
}

// Upper bound of the planner's item count: a q tile with T KV tiles becomes at most T / L + 1
// items, and the planner's chunk length L is at least (sum of T) x hkv / (kItemsPerSlot x slots); the
// remainder round adds fewer than slots / hkv.  The prefix of a group (or of a slice of one, whose tiles
// are in that sum too) adds at most one item per sequence beyond that.
int32_t item_bound(const WorkspaceLayout& w, int hkv, int slots, bool groups) {
  int64_t b = w.max_tiles;
  if (may_cut(w, hkv, slots)) b += (int64_t)kItemsPerSlot * slots / hkv + 1;
  if (groups) b += w.batch;
  return (int32_t)(b < w.max_items ? b : w.max_items);
}

mc_status check_attn_shape(const mc_pool_desc* pool, int32_t num_q_heads, int32_t batch,
                           int32_t total_q, int* G_out) {
  mc_status st = mc::check_pool(pool);
  if (st != MC_OK) return st;
  if (num_q_heads <= 0 || batch < 0 || total_q < 0) return MC_ERR_INVALID;
  if (num_q_heads % pool->num_kv_heads != 0) return MC_ERR_UNSUPPORTED;
  const int G = num_q_heads / pool->num_kv_heads;
  if (G != 1 && G != 2 && G != 4 && G != 8) return MC_ERR_UNSUPPORTED;
  *G_out = G;
  return MC_OK;
}

mc_status plan_impl(const mc_pool_desc* pool, int32_t num_q_heads, int32_t batch,
                    int32_t total_q, const int32_t* cu_q, const int32_t* begin,
                    const int32_t* page_table, const int32_t* cu_pages, int32_t ahead_tokens,
                    void* workspace, size_t workspace_bytes, int32_t part_limit, void* stream) {
  if (ahead_tokens < 0 || ahead_tokens > (1 << 20)) return MC_ERR_RANGE;
  int G = 0;
  mc_status st = check_attn_shape(pool, num_q_heads, batch, total_q, &G);
  if (st != MC_OK) return st;
  if (!workspace || !mc::aligned16(workspace)) return MC_ERR_INVALID;
  const int tile_tokens = kBM / G;
  const WorkspaceLayout w =
      workspace_layout(batch, total_q, tile_tokens, num_q_heads, pool->num_kv_heads, part_limit);
  if (workspace_bytes < w.total) return MC_ERR_INVALID;
  if (batch > 0 && (!cu_q || !begin || !page_table || !cu_pages)) return MC_ERR_INVALID;
  if (batch == 0) {   // nothing to plan: a header with an empty work list
    if (!cu_q || !cu_pages) return MC_ERR_INVALID;
  }
  char* ws = static_cast<char*>(workspace);
  PlanArgs a;
  a.cu_q = cu_q;
  a.begin = begin;
  a.page_table = page_table;
  a.cu_pages = cu_pages;
  a.hdr = reinterpret_cast<PlanHeader*>(ws);
  a.cu_tiles = reinterpret_cast<int32_t*>(ws + w.cu_tiles);
  a.items = reinterpret_cast<ItemRec*>(ws + w.items);
  a.arrivals_end = reinterpret_cast<uint32_t*>(ws + w.part_lse) + (size_t)w.part_cap * num_q_heads;
  a.batch = batch;
  a.total_q = total_q;
  a.tile_tokens = tile_tokens;
  a.num_pages = pool->num_pages;
  a.max_tiles = w.max_tiles;
  a.hq = num_q_heads;
  a.hkv = pool->num_kv_heads;
  a.slots = device_slots(1);
  if (a.slots <= 0) return MC_ERR_HIP;
  const bool wide = wide_tiles_allowed(batch, total_q, G, pool->num_kv_heads);
  a.wide_tile_tokens = wide ? 2 * tile_tokens : 0;
  a.slots_wide = device_slots(2);
  a.allow_groups = may_group(w, total_q, tile_tokens);
  a.max_items = item_bound(w, a.hkv, a.slots, a.allow_groups);
  a.merges = reinterpret_cast<MergeRec*>(a.items + a.max_items);
  a.max_merges = (int32_t)((ws + w.part_lse - (char*)a.merges) / sizeof(MergeRec));
  a.part_cap = w.part_cap;
  a.ahead = ahead_tokens;
  // (few sequences only: the page-id checks and the table comparisons of shared prefixes go
  // a wavefront per sequence or pair and want the wavefronts of the large workgroup)
  hipStream_t hs = static_cast<hipStream_t>(stream);
  if (may_narrow(batch, total_q, G, a.hkv, a.slots))
    hipLaunchKernelGGL((plan_kernel<kPlanThreadsSmall, true>), dim3(1), dim3(kPlanThreadsSmall), 0, hs, a);
  else if (batch <= 16 && w.max_tiles <= 8 * kPlanThreadsSmall)
    hipLaunchKernelGGL((plan_kernel<kPlanThreadsSmall, false>), dim3(1), dim3(kPlanThreadsSmall), 0, hs, a);
  else
    hipLaunchKernelGGL((plan_kernel<kPlanThreads, false>), dim3(1), dim3(kPlanThreads), 0, hs, a);
  if (batch > kValidateInPlan)
    hipLaunchKernelGGL(validate_pages_kernel, dim3((batch + 3) / 4), dim3(256), 0, hs, a);
  return mc::launch_status();
}


mc_status attn_impl(const mc_pool_desc* pool, int32_t layer, const void* q, int32_t num_q_heads,
                    int32_t batch, int32_t total_q, const int32_t* cu_q, const int32_t* begin,
                    const int32_t* page_table, const int32_t* cu_pages, float sm_scale, void* out,
                    float* lse, void* workspace, size_t workspace_bytes, int32_t part_limit,
                    void* stream) {
  int G = 0;
  mc_status st = check_attn_shape(pool, num_q_heads, batch, total_q, &G);
  if (st != MC_OK) return st;
  if (layer < 0 || layer >= pool->num_layers) return MC_ERR_RANGE;
  if (!(sm_scale >= 0.f) || !isfinite(sm_scale)) return MC_ERR_INVALID;
  if (batch == 0 || total_q == 0) return MC_OK;
  if (!q || !out || !lse || !cu_q || !begin || !page_table || !cu_pages || !workspace)
    return MC_ERR_INVALID;
  if (!mc::aligned16(q) || !mc::aligned16(out) || !mc::aligned16(workspace) ||
      (reinterpret_cast<uintptr_t>(lse) & 3u))
    return MC_ERR_INVALID;
  const int tile_tokens = kBM / G;
  const WorkspaceLayout w =
      workspace_layout(batch, total_q, tile_tokens, num_q_heads, pool->num_kv_heads, part_limit);
  if (workspace_bytes < w.total) return MC_ERR_INVALID;
  const int slots = device_slots(1);
  if (slots <= 0) return MC_ERR_HIP;
  const bool groups = may_group(w, total_q, tile_tokens);
  const int32_t max_items = item_bound(w, pool->num_kv_heads, slots, groups);
  const int64_t blocks = (int64_t)max_items * pool->num_kv_heads;
  if (blocks > 0x7fffffffll) return MC_ERR_UNSUPPORTED;
  char* ws = static_cast<char*>(workspace);
  AttnArgs a;
  a.pool_layer = static_cast<const char*>(pool->base) + layer * mc::layer_stride_bytes(pool);
  a.q = static_cast<const char*>(q);
  a.out = static_cast<char*>(out);
  a.lse = lse;
  a.begin = begin;
  a.page_table = page_table;
  a.hdr = reinterpret_cast<const PlanHeader*>(ws);
  a.items = reinterpret_cast<const ItemRec*>(ws + w.items);
  a.merges = reinterpret_cast<const MergeRec*>(a.items + max_items);
  a.part_lse = reinterpret_cast<float*>(ws + w.part_lse);
  a.part_o = reinterpret_cast<float*>(ws + w.part_o);
  a.part_cap = w.part_cap;
  a.units = slots / 2;
  a.num_pages = pool->num_pages;
  a.hkv = pool->num_kv_heads;
  a.hq = num_q_heads;
  a.batch = batch;
  a.total_q = total_q;
  // (q tiles there are at least.  A batch of rows that are all few has no trees.)
  const int64_t tiles = (int64_t)(w.max_tiles - batch) * pool->num_kv_heads;
  const bool trees = w.part_cap > 0 && total_q > batch && (int64_t)total_q * G > kFlatRows;
  a.behind = groups && !groups_in_launch(batch, total_q) ? kGroupsBehind : 0;
  if (trees && a.behind != 0 && trees_behind(tiles, slots)) a.behind |= kTreesBehind;
  a.scale = sm_scale > 0.f ? sm_scale : 1.0f / sqrtf((float)mc::kHeadDim);
  a.scale_log2 = a.scale * 1.4426950408889634f;
  dim3 grid((unsigned)blocks);
  hipStream_t hs = static_cast<hipStream_t>(stream);
  // many sequences for the number of q tiles: a good share of the tiles is short
  const int mode = may_narrow(batch, total_q, G, pool->num_kv_heads, slots) ? kNarrowTiles
                   : 4ll * batch >= w.max_tiles - batch                     ? kGated
                                                                            : kPlain;
  st = pool->dtype == MC_F16 ? launch_attn<_Float16>(G, mode, 1, grid, hs, a)
                             : launch_attn<__bf16>(G, mode, 1, grid, hs, a);
  if (st == MC_OK && wide_tiles_allowed(batch, total_q, G, pool->num_kv_heads)) {
    // the plan may be one of wide q tiles (fewer items than the grid's bound, which holds for
    // either width): that kernel, too; the one the plan was not made for finds the other tile
    // size in the header and returns
    st = pool->dtype == MC_F16 ? launch_attn<_Float16>(G, kPlain, 2, grid, hs, a)
                               : launch_attn<__bf16>(G, kPlain, 2, grid, hs, a);
  }
  if (st != MC_OK || a.behind == 0) return st;
  const int rows = std::min((total_q + batch - 1) / batch * G, kBM), per_block = kThreads / 32;
  const int row_blocks = (rows + per_block - 1) / per_block;
  const int64_t all = (int64_t)w.max_tiles * row_blocks * pool->num_kv_heads;
  const dim3 mgrid((unsigned)std::min<int64_t>(all, slots));
  if (pool->dtype == MC_F16) launch_merge<_Float16>(G, mgrid, row_blocks, hs, a);
  else launch_merge<__bf16>(G, mgrid, row_blocks, hs, a);
  return mc::launch_status();
}


// ---- scratch of the entry point that allocates nothing ---------------------------------
// The attention workspace (work list, partial rows) of mc_prefix_prefill_attn_noalloc lives in
// this array; every GPU the library runs on holds its own copy until the process ends.
constexpr size_t kScratchBytes = size_t(8) << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

// Device address of the current device's copy of `scratch` (in host code the array's name is
// only a handle for this look-up, never an address a kernel may use).  Looked up once per device.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};

mc_status scratch_of_current_device(void** ptr_out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return MC_ERR_HIP;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return MC_ERR_HIP;
    g_scratch_ptr[dev] = ptr;
  }
  *ptr_out = g_scratch_ptr[dev];
  return MC_OK;
}

}  // namespace

extern "C" {

size_t mc_attn_workspace_size(int32_t batch, int32_t total_q, int32_t num_q_heads,
                              int32_t num_kv_heads) {
  if (batch < 0 || total_q < 0 || num_q_heads <= 0 || num_kv_heads <= 0) return 0;
  if (num_q_heads % num_kv_heads != 0) return 0;
  const int G = num_q_heads / num_kv_heads;
  if (G != 1 && G != 2 && G != 4 && G != 8) return 0;
  return workspace_layout(batch, total_q, kBM / G, num_q_heads, num_kv_heads).total;
}

mc_status mc_attn_plan(const mc_pool_desc* pool, int32_t num_q_heads, int32_t batch,
                       int32_t total_q, const int32_t* cu_q, const int32_t* begin,
                       const int32_t* page_table, const int32_t* cu_pages, void* workspace,
                       size_t workspace_bytes, void* stream) {
  return mc_attn_plan_ahead(pool, num_q_heads, batch, total_q, cu_q, begin, page_table, cu_pages,
                            0, workspace, workspace_bytes, stream);
}

mc_status mc_attn_plan_ahead(const mc_pool_desc* pool, int32_t num_q_heads, int32_t batch,
                             int32_t total_q, const int32_t* cu_q, const int32_t* begin,
                             const int32_t* page_table, const int32_t* cu_pages,
                             int32_t ahead_tokens, void* workspace, size_t workspace_bytes,
                             void* stream) {
  return plan_impl(pool, num_q_heads, batch, total_q, cu_q, begin, page_table, cu_pages,
                   ahead_tokens, workspace, workspace_bytes, -1, stream);
}

mc_status mc_attn_plan_check(const void* workspace, void* stream) {
  if (!workspace) return MC_ERR_INVALID;
  PlanHeader h;
  hipStream_t hs = static_cast<hipStream_t>(stream);
  if (hipMemcpyAsync(&h, workspace, sizeof(h), hipMemcpyDeviceToHost, hs) != hipSuccess)
    return MC_ERR_HIP;
  if (hipStreamSynchronize(hs) != hipSuccess) return MC_ERR_HIP;
  if (h.magic != kPlanMagic) return MC_ERR_INVALID;
  return static_cast<mc_status>(h.err);
}

mc_status mc_prefix_prefill_attn(const mc_pool_desc* pool, int32_t layer, const void* q,
                                 int32_t num_q_heads, int32_t batch, int32_t total_q,
                                 const int32_t* cu_q, const int32_t* begin,
                                 const int32_t* page_table, const int32_t* cu_pages,
                                 float sm_scale, void* out, float* lse, void* workspace,
                                 size_t workspace_bytes, void* stream) {
  return attn_impl(pool, layer, q, num_q_heads, batch, total_q, cu_q, begin, page_table, cu_pages,
                   sm_scale, out, lse, workspace, workspace_bytes, -1, stream);
}

mc_status mc_prefix_prefill_attn_noalloc(const mc_pool_desc* pool, int32_t layer, const void* q,
                                         int32_t num_q_heads, int32_t batch, int32_t total_q,
                                         const int32_t* cu_q, const int32_t* begin,
                                         const int32_t* page_table, const int32_t* cu_pages,
                                         float sm_scale, void* out, float* lse, void* stream) {
  int G = 0;
  mc_status st = check_attn_shape(pool, num_q_heads, batch, total_q, &G);
  if (st != MC_OK) return st;
  // the work list alone must fit; what is left holds partial rows (64-byte item record, LSE
  // and O per row and q head), fewer than the caller-workspace variant may ask for
  const int tile_tokens = kBM / G;
  const WorkspaceLayout fixed =
      workspace_layout(batch, total_q, tile_tokens, num_q_heads, pool->num_kv_heads, 0);
  if (fixed.total + 4096 > kScratchBytes) return MC_ERR_RANGE;
  const size_t per_row = sizeof(ItemRec) + sizeof(float) * (size_t)num_q_heads * (mc::kHeadDim + 1);
  int32_t part_limit = (int32_t)((kScratchBytes - fixed.total - 4096) / per_row);
  while (part_limit > 0 &&
         workspace_layout(batch, total_q, tile_tokens, num_q_heads, pool->num_kv_heads, part_limit)
                 .total > kScratchBytes)
    --part_limit;
  void* ws = nullptr;
  st = scratch_of_current_device(&ws);
  if (st != MC_OK) return st;
  st = plan_impl(pool, num_q_heads, batch, total_q, cu_q, begin, page_table, cu_pages, 0, ws,
                 kScratchBytes, part_limit, stream);
  if (st != MC_OK) return st;
  return attn_impl(pool, layer, q, num_q_heads, batch, total_q, cu_q, begin, page_table, cu_pages,
                   sm_scale, out, lse, ws, kScratchBytes, part_limit, stream);
}

}  // extern "C"
