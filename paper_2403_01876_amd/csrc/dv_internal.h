// Internal launch descriptors shared by the host dispatch (dv_api.cpp) and
// the kernels (dv_kernels.hip).  Units are 16 bytes throughout: every cache
// and wire address handled here is a multiple of 16 bytes, which lets each
// lane move one 128-bit word per access.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dv {

// Sequences of an ordinary launch: one per lane of a 64-wide wavefront.  (Larger
// batches go kSeqMany to a launch.)
constexpr int kSeqPerLaunch = 64;
constexpr int kThreads = 256;

// Workgroups in x that a launch has fewer than: a grid's lanes are counted in 32
// bits.  (A test's build sets a small limit, so that small shapes take the paths
// of slabs of 128 GB; more than the sequences of a call.)
#ifdef DV_MAX_GROUPS
constexpr int64_t kMaxGroups = DV_MAX_GROUPS;
#else
constexpr int64_t kMaxGroups = (1ll << 32) / kThreads;
#endif

enum Dir : int { kPack = 0, kUnpack = 1 };

// Division by a launch constant d >= 1, exact for 0 <= n < 2^31: with l =
// ceil(log2 d) and m = ceil(2^(31 + l) / d) (below 2^32), n / d = n * m >> (31
// + l) (Granlund and Montgomery, "Division by invariant integers using
// multiplication", PLDI 1994).  Doubling n first keeps d = 1 in the same form.
struct FastDiv {
  uint32_t m, l;
  __host__ __device__ uint32_t div(uint32_t n) const {
#if defined(__HIP_DEVICE_COMPILE__)
    return __umulhi(n << 1, m) >> l;
#else
    return (uint32_t)(((uint64_t)(n << 1) * m) >> 32) >> l;
#endif
  }
};
inline FastDiv fast_div(uint32_t d) {
  FastDiv f{0, 0};
  while ((1ull << f.l) < d) ++f.l;
  f.m = (uint32_t)(((1ull << (31 + f.l)) + d - 1) / d);
  return f;
}

// The sequences of one launch (N of them at most: 64, or 256 for larger
// batches), with the prefixes that place them computed on the host: a
// workgroup finds its sequence with one ballot per 64 entries instead of
// scanning the counts.
constexpr int kSeqMany = 256;

// 16-byte units per lane of the kernel for several tokens in split-key caches.
constexpr int kRowsUnroll = 2;
template <int N>
struct SeqTable {
  int32_t item[N];     // work items of all earlier sequences; INT32_MAX past the last
  int32_t tok[N + 1];  // tokens of all earlier sequences
  int32_t t0[N];       // first token of each sequence's range
};

struct SeqRanges {
  int32_t t0[kSeqPerLaunch];  // first token of each sequence's range
  int32_t n[kSeqPerLaunch];   // tokens in the range (0 = sequence skipped)
};

// Slab = one (layer, K|V) half of the cache; grid row y handles cache slab
// slab0 + y, whose data sits in wire slab y.
struct SlabMap {
  int32_t slab0, pad;
  int64_t w_slab;  // wire units per slab: N * heads * du
};

// A launch's (tile, slab) grid, dealt so that each of the chip's 8 XCDs takes
// one contiguous eighth of it, or (on = 0) left in the hardware's order.
struct Deal {
  uint32_t tiles;    // per slab (the grid's width)
  uint32_t q, r;     // eighths of the grid: r of q + 1 items, the others of q
  uint32_t on;
  FastDiv d_tiles;
};
inline Deal deal_of(int64_t tiles, int64_t slabs, bool eighths) {
  const int64_t total = tiles * slabs;
  const bool on = eighths && total < (1ll << 31);
  return Deal{(uint32_t)tiles, on ? (uint32_t)(total / 8) : 0, (uint32_t)(total % 8), on,
              fast_div((uint32_t)tiles)};
}

// Dense runs: for each (sequence, head) the range is one contiguous run of
// n*du units in the cache and in the wire.
template <int N>
struct DenseRunArgs {
  void* cache;     // microbatch base, advanced to this launch's first sequence
  void* wire;      // wire base advanced to this launch's first sequence
  int64_t s_slab;  // cache units per slab
  int64_t s_b;     // cache units per sequence
  int64_t s_h;     // cache units per head
  SlabMap m;
  int32_t du;      // units per token (head_dim * elem_bytes / 16)
  int32_t heads;
  Deal deal;
  SeqTable<N> s;
};

// Paged blocks.  A slab of the pool is one array of units in (block, head,
// token, group) order; a tile is kPagedTile consecutive units of it, or, in
// table order, of the array its blocks would form if each sequence's blocks
// stood in the table's order.  So a tile's pool side is contiguous up to block
// boundaries and every lane holds a unit whatever the block's size.  With
// `owner` set (pool order) a block's sequence comes from the owner map.
template <int N>
struct PagedArgs {
  void* pool;
  void* wire;            // contiguous buffer advanced to this launch's first sequence
  const int32_t* bt;     // rows of this launch's sequences [nseq][max_blocks]
  const int32_t* owner;  // pool order: [num_blocks] owner map, else null
  int64_t s_slab;        // pool units per slab (NB * heads * bs * du)
  int64_t s_blk;         // pool units per block (heads * bs * du)
  SlabMap m;
  int32_t ub;            // pool units per head in a block (bs * du)
  int32_t du, heads, nseq;
  int32_t num_blocks, max_blocks;
  int32_t tiles;         // tiles per slab (the grid's width)
  int32_t steps;         // wide launches: tiles a workgroup takes one after another
  FastDiv d_ub, d_heads, d_bs, d_max, d_tiles;
  SeqTable<N> s;
};
static_assert(sizeof(PagedArgs<kSeqMany>) <= 3584, "arguments stay well under 4 KB");

// Sequences a pool-order stream-in covers.
constexpr int kPoolSeqMax = kSeqMany;

// Owner map of a paged table over the streamed ranges: owner[blk] =
// b * max_blocks + j for each entry (b, j) whose logical block j holds a
// streamed token of sequence b and whose block blk is in [0, num_blocks);
// -1 for every other block.  Small tables: one launch (OwnerMapArgs).  Large
// ones: one clearing launch and one launch per group of up to 64 sequences, b0
// being the group's first sequence.
struct OwnerArgs {
  int32_t* owner;
  const int32_t* bt;
  int32_t nseq, block_size, num_blocks, max_blocks;
  int32_t b0, pad;  // index of the launch's first sequence
  SeqRanges r;
};

// The whole map in one launch: a workgroup owns kOwnerSpan blocks of the pool
// and looks through every table entry of the ranges for them, 64 entries (a
// chunk, s.item counts them) to a wave.
template <int N>
struct OwnerMapArgs {
  int32_t* owner;
  const int32_t* bt;
  int32_t chunks, num_blocks, max_blocks, pad;
  FastDiv d_bs;
  SeqTable<N> s;
};
constexpr int kOwnerSpan = 512;
constexpr int kOwnerThreads = 1024;
// One launch is used while its chunks are at most this many for each launch that
// the other way takes, one to clear and one per 64 sequences: every workgroup
// reads every entry, so the launches saved are paid for in large pools.  A
// pool-order stream-in of one layer, one head, graph-replayed, several launches
// and one: up to 64 sequences (two launches) 544 blocks (32 chunks) 6.7 and 5.7
// us, 4600 blocks (72) 17.6 and 16.5, 19200 blocks (320) 55.2 and 57.3; 100
// sequences (three) 400 chunks 12.1 and 14.8; 150 (four) 450 chunks 14.5 and 15.7;
// 200 (five) 400 chunks 15.7 and 15.0; 220 (five) 440 chunks 16.6 and 15.7; 256
// (five) 512 chunks 16.6 and 16.8, 768 chunks 20.5 and 24.9.
constexpr int kOwnerChunks = 96;

// Short runs (decode-step increments of one or a few tokens per sequence):
// the 16-byte units of a slab in wire order, (sequence, head, token, group),
// spread evenly over the lanes, so that none idles the way it would in a tile
// sized for long runs.  A row is one token of one head: du units.  Only the
// sequences with a token in the range are listed; unit g of a row sits at
// cache offset sequence or block + head * s_h + token * s_tok[half] + g *
// s_e[half], half 0 for key slabs and 1 for value slabs (a split-key cache's
// differ), and both halves go in one launch.
template <int N>
struct RowArgs {
  void* cache;
  void* wire;          // contiguous buffer advanced to this launch's first sequence
  const int32_t* bt;   // paged only
  int64_t s_slab;
  int64_t s_b;         // dense: units per sequence; paged: units per block
  int64_t s_h;         // units per head
  int64_t s_tok[2], s_e[2];
  SlabMap m;
  int32_t total;       // units per slab of this launch (below 2^31)
  int32_t du, heads;
  int32_t paged, block_size, num_blocks, max_blocks;
  int32_t n;           // tokens of every sequence, where they are equal
  int32_t tile;        // rows per workgroup (split_rows_kernel)
  FastDiv d_du, d_heads, d_seq, d_n, d_bs, d_tile;  // d_seq: heads * n
  int32_t tok[N + 1];  // ragged: tokens of all earlier sequences; INT32_MAX past the last
  int32_t t0[N];       // first token of each sequence's range
  int32_t seq[N];      // its index in the cache
};
static_assert(sizeof(RowArgs<kSeqMany>) <= 3584, "arguments stay well under 4 KB");

// Split-key caches, long runs: a tile is a.tile tokens of one (sequence, head);
// key slabs go through LDS, value slabs straight across, in one launch.  Where a
// head's groups start on lines of 8 tokens (line_mask 7), tiles end on them too:
// a run's first tile is shorter by the tokens its start lies past one.
template <int N>
struct SplitArgs {
  void* cache;
  void* wire;            // contiguous buffer advanced to this launch's first sequence
  int64_t s_slab, s_b, s_h;  // as dense
  SlabMap m;
  int32_t du;            // 16-byte groups per token, <= kKsplitMaxDu
  int32_t heads, b0;
  int32_t seq_cap;       // S: units between consecutive groups of one head
  int32_t tile;          // tokens per tile (a multiple of 8)
  int32_t line0, line_mask;  // token t lies (line0 + t) & line_mask past a line's start
  Deal deal;
  FastDiv d_du, d_tile;
  SeqTable<N> s;
};

// Tokens per tile: whole 128-byte lines of a key slab (8 tokens of a group) in
// two units per lane, six or eight.  Six where two would leave more than a fifth
// of the lanes idle (17 and 22-25 groups per token: 24 and 16 tokens fill 69 to 80
// %).  37 layers of 12 heads x 96 x 4 bytes, 0.76 GB: 259 and 269 us out and in
// with six, 261 and 283 with two, 263 and 281 with four.
inline int32_t split_tile(int64_t du, int units) { return (int32_t)(units * kThreads / du & ~7); }
inline int split_units(int64_t du) { return 5 * split_tile(du, 2) * du >= 4 * 2 * kThreads ? 2 : 6; }
// Eight instead of two for a stream-in from this many groups per token on where
// max_seq is not whole lines, so that every tile ends inside some (run_split has
// the rest of the rule).  Two and eight, 20 heads, launches of 300 MB: 32 groups,
// 50-62 tokens 120 and 109 us, 20-30 tokens 152 and 134, 0-47 tokens 145 and 135 (as
// good as two when they fill less than a third), 300-1100 tokens 102 and 98, but
// 70-75 tokens, a second tile for the last few, 115 and 120; 20 groups, 36-50 tokens
// 125 and 119; 16 groups, 300-1100 tokens 137 and 137.  Smaller launches: 20 MB 9.1
// and 8.3, 9 MB 5.5 and 5.7, 3 MB 3.0 and 3.6.
constexpr int64_t kSplitEightDu = 20, kSplitEightMin = 1 << 20;
constexpr size_t kSplitLdsFor4 = 39 * 1024;  // 4 per CU fit in 160 KB, 5 do not

// Cache-to-cache copy of the same logical positions between two dense caches
// (device slot <-> pinned host mirror) for narrow rows: rows as in RowArgs,
// with a place in each cache.
template <int N>
struct CopyArgs {
  void* src;
  void* dst;
  int64_t s_slab, s_b, s_h;  // source strides (units); token stride du
  int64_t d_slab, d_b, d_h;  // destination strides (units)
  int32_t slab0;             // grid row y copies slab slab0 + y
  int32_t total;             // units per slab of this launch (below 2^31)
  int32_t du, heads;
  FastDiv d_du, d_heads;
  int32_t tok[N + 1];        // as RowArgs
  int32_t t0[N];
  int32_t seq[N];
};
constexpr int kCopyUnroll = 1;

constexpr int kKsplitMaxDu = 32;

// Launchers (dv_kernels.hip).  Each returns the hipError_t of its launch.
template <int N>
hipError_t launch_dense_runs(int dir, const DenseRunArgs<N>& a, uint32_t nslabs, hipStream_t s);
// `wide`: some tile's first unit, or the number of the grid's workgroups, may
// pass 2^31 (steps is 1 otherwise).
template <int N>
hipError_t launch_paged(int dir, const PagedArgs<N>& a, bool wide, uint32_t nslabs,
                        hipStream_t s);
// Sets every entry of the owner map to -1.
hipError_t launch_owner_clear(const OwnerArgs& a, hipStream_t s);
// Fills the owner map from the table for sequences [b0, b0 + nseq).
hipError_t launch_owner_build(const OwnerArgs& a, hipStream_t s);
template <int N>
hipError_t launch_owner_map(const OwnerMapArgs<N>& a, hipStream_t s);
// Counts, per pool block, the table entries over the ranges of sequences
// [b0, b0 + nseq) that map to it, into `a.owner` (int32 counts), clearing
// the counts first when `clear` is set.
hipError_t launch_block_claims(const OwnerArgs& a, bool clear, hipStream_t s);
// `even`: every sequence has a.n tokens.
template <int N>
hipError_t launch_rows(int dir, bool even, const RowArgs<N>& a, uint32_t nslabs, hipStream_t s);
template <int N>
hipError_t launch_split_rows(int dir, const RowArgs<N>& a, uint32_t nslabs, hipStream_t s);
template <int N>
hipError_t launch_split(int dir, const SplitArgs<N>& a, uint32_t nslabs, hipStream_t s);
template <int N>
hipError_t launch_copy(const CopyArgs<N>& a, uint32_t nslabs, hipStream_t s);

// Units each dense-run workgroup moves (tiles are counted on the host with
// the same constant).  Two 16-byte units per lane (8 KB per workgroup) keeps
// register use low enough for full occupancy; measured on MI355X against 1,
// 3, 4, 8 and 16 units per lane on the OPT-13B stage shape.
constexpr int kDenseUnroll = 2;
constexpr int kDenseTile = kThreads * kDenseUnroll;

// 16-byte units per paged tile: two per lane, 8 KB of one pool slab.
constexpr int kPagedUnroll = 2;
constexpr int kPagedTile = kThreads * kPagedUnroll;

// Pool-order scatters deal their (tile, slab) grid to the 8 XCDs in chunks of
// this many consecutive tiles (8 pool blocks of one slab at 8 heads; 256 KB for
// the LLaMA-2-70B pool).  Measured on MI355X on that pool against the hardware's
// round-robin dealing, contiguous eighths and chunks of 8, 16, 48 and 64 tiles.
constexpr int kPoolChunk = 32;
// The same for table-order launches whose tiles cross blocks.  80 layers of one
// head, 1-byte cache, gather and scatter: round robin 903 and 990 us, chunks of
// 4 907 and 996, of 16 890 and 969, of 64 887 and 968, of 256 898 and 972,
// eighths 936 and 1013; launches of 400 MB do not tell them apart.
constexpr int kTableChunk = 64;

}  // namespace dv
