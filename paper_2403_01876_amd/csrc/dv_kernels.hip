// Pack / unpack kernels for gfx950.  Pure data movement: every lane moves
// 16-byte words with nontemporal global loads and stores (the data is
// streamed once, so it should not displace L2/MALL contents; only the swap
// kernel's stores are ordinary ones), no arithmetic touches the payload and no
// MFMA is involved.
//
// Work resolution: a launch covers at most 64 sequences, one per lane of a
// wavefront, or 256, four per lane.  Their ranges travel by value in the kernel
// arguments with the prefixes of their tile and token counts, so nothing is
// copied to the device before a launch; a ballot of "prefix <= my tile" gives
// the workgroup's sequence.  Divisions by extents that a launch shares are
// multiplications (FastDiv).
#include "dv_internal.h"

namespace dv {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ u32x4 ld_nt(const u32x4* p) { return __builtin_nontemporal_load(p); }
__device__ __forceinline__ void st_nt(u32x4 v, u32x4* p) { __builtin_nontemporal_store(v, p); }

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }

// The sequence that holds work item `item` of a launch, uniform over the
// wavefront: every lane compares the prefixes of its share of the sequences,
// and the count of prefixes at or below the item names the sequence (empty
// sequences share their successor's prefix, so the last one counted has it).
struct Seq {
  int b, k;      // index in the launch; the item's index in the sequence
  int t0, n, p;  // first token, tokens, tokens of earlier sequences
};
template <int N>
__device__ __forceinline__ Seq find_seq(const SeqTable<N>& s, int item) {
  const int lane = lane_id();
  Seq q;
  if constexpr (N == 64) {
    const int first = s.item[lane], t0 = s.t0[lane], p = s.tok[lane], p1 = s.tok[lane + 1];
    q.b = __popcll(__ballot(first <= item)) - 1;
    q.k = item - __builtin_amdgcn_readlane(first, q.b);
    q.t0 = __builtin_amdgcn_readlane(t0, q.b);
    q.p = __builtin_amdgcn_readlane(p, q.b);
    q.n = __builtin_amdgcn_readlane(p1, q.b) - q.p;
  } else {
    int below = 0;
#pragma unroll
    for (int i = 0; i < N / 64; ++i) below += __popcll(__ballot(s.item[i * 64 + lane] <= item));
    q.b = below - 1;
    q.k = item - s.item[q.b];
    q.t0 = s.t0[q.b];
    q.p = s.tok[q.b];
    q.n = s.tok[q.b + 1] - q.p;
  }
  return q;
}

// Workgroup IDs are dealt round-robin to the chip's 8 XCDs (each with its
// own L2).  The bulk kernels re-deal the linearised (tile, slab) grid so each
// XCD streams a contiguous range of it: workgroup `lin` runs on XCD lin % 8
// and takes item lin / 8 of that XCD's range; XCD x owns q items (one more if x
// < r) starting at x * q + min(x, r).  The map is a bijection on the grid
// whatever order the hardware actually deals workgroups in; on MI355X it lifts
// the dense copy from 74 % to 77-79 % of HBM peak.  (The paged kernels do not
// use it; see xcd_chunk.)
__device__ __forceinline__ void xcd_tile(const Deal& d, uint32_t* tile, uint32_t* slab) {
  *tile = blockIdx.x;
  *slab = blockIdx.y;
  if (!d.on) return;
  const uint32_t lin = blockIdx.x + blockIdx.y * d.tiles, x = lin % 8;
  const uint32_t t = x * d.q + min(x, d.r) + lin / 8;
  *slab = d.d_tiles.div(t);
  *tile = t - *slab * d.tiles;
}

// The linearised (tile, slab) grid dealt to the XCDs in chunks of C consecutive
// items.  Workgroup `lin` runs on XCD lin % 8 and takes item (lin / 8) % C of
// that XCD's (lin / 8) / C-th chunk; round r gives chunk 8r + x to XCD x.
// Items past the last whole round keep their place.  A bijection on [0, total),
// whatever order the hardware actually deals workgroups in.  On MI355X chunks
// of 32 lift the LLaMA-2-70B pool-order scatter from 75 % to 77 % of HBM peak,
// where contiguous eighths (as xcd_tile) cost it 2 points and cost the
// table-order gather 6.
template <typename U>
__device__ __forceinline__ U xcd_chunk(U lin, U total, U C) {
  const U full = total / (8 * C) * (8 * C);
  if (lin >= full) return lin;
  const U x = lin % 8, k = lin / 8;
  return ((k / C) * 8 + x) * C + k % C;
}

// ---------------------------------------------------------------------------
// Dense runs: grid (tiles_per_slab, nslabs); a tile is kDenseTile units of
// one (sequence, head) run.  Bound by HBM for whole prompts (6.2 TB/s, a plain
// copy 6.5); launches of tens of microseconds also by how soon the first loads
// leave: with the sequence found by two wavefront scans and the grid dealt by
// 64-bit divisions, 402 instructions before them instead of about 150, one
// layer of the OPT-13B stage's prompts (126 MB) took 44.2 us instead of 42.6,
// 410 KB 2.5 us instead of 2.0.
// ---------------------------------------------------------------------------
template <int D, int N>
__global__ void __launch_bounds__(kThreads) dense_runs_kernel(DenseRunArgs<N> a) {
  uint32_t tile, y;
  xcd_tile(a.deal, &tile, &y);
  const Seq q = find_seq(a.s, tile);
  const int run = q.n * a.du;
  const uint32_t tpr = (run + kDenseTile - 1) / kDenseTile;
  const uint32_t h = (uint32_t)q.k / tpr, k = (uint32_t)q.k - h * tpr;

  u32x4* cache = (u32x4*)a.cache + (int64_t)(a.m.slab0 + y) * a.s_slab + (int64_t)q.b * a.s_b +
                 (int64_t)h * a.s_h + (int64_t)q.t0 * a.du + (int64_t)k * kDenseTile;
  u32x4* wire = (u32x4*)a.wire + (int64_t)y * a.m.w_slab +
                (int64_t)q.p * ((int64_t)a.heads * a.du) + (int64_t)h * run +
                (int64_t)k * kDenseTile;
  const u32x4* src = (D == kPack) ? cache : wire;
  u32x4* dst = (D == kPack) ? wire : cache;
  const int count = min(kDenseTile, run - (int)k * kDenseTile);

  // Loads carry no per-lane guard (a lane past the tile's end re-reads the
  // tile's last unit), so they issue back to back with a single wait; a
  // guarded load would make the compiler wait after every one.
  u32x4 v[kDenseUnroll];
#pragma unroll
  for (int i = 0; i < kDenseUnroll; ++i)
    v[i] = ld_nt(src + min(i * kThreads + (int)threadIdx.x, count - 1));
#pragma unroll
  for (int i = 0; i < kDenseUnroll; ++i) {
    const int idx = i * kThreads + threadIdx.x;
    if (idx < count) st_nt(v[i], dst + idx);
  }
}

// ---------------------------------------------------------------------------
// Paged blocks: grid (tiles_per_slab, nslabs); a tile is kPagedTile units of
// the slab's (block, head, token, group) order (see PagedArgs).
//
// Table order (POOL false): the blocks stand in (sequence, logical block)
// order and are found through the table, so consecutive workgroups touch
// consecutive wire bytes.  Pool order (unpack only): they stand as in the
// pool and the owner map names each one's (sequence, logical block), so
// consecutive workgroups write consecutive pool bytes -- on MI355X writes
// scattered by a random table cost more than reads scattered the same way.
//
// Bound by HBM once a workgroup's fixed cost (dispatch, its sequence, the
// table entry) is spread over a whole tile.  Tiles of two heads of one block
// left that cost on 2 KB for one KV head of a 1-byte cache (80 layers, 64
// sequences of 128-4096 tokens, 2.77 GB): 2320 and 2350 us a gather and a
// scatter, 2.4 TB/s; with tiles of 512 units across blocks 910 and 990 us, 6.1
// and 5.6 TB/s.  Where a tile was whole before, the LLaMA-2-70B pool (eight
// heads of a 2-byte cache, 5.54 GB), nothing is gained in use: a gather and a
// pool-order scatter after each other take 3635 us, 3643 before, within noise
// (each replayed by itself 1784 and 1759 us, 1827 and 1776 before).
//
// ONE: a tile never leaves its block (the block is a multiple of the tile),
// so block, table entry and sequence are uniform over the workgroup.  WIDE:
// unit numbers may pass 2^31, and a workgroup may take several tiles; kept
// apart so that the ordinary kernels run straight down, with their arguments
// fetched together.  TWO: blocks of a wave's units and more, looked up by the wave
// (launch_paged has the rule).
// ---------------------------------------------------------------------------
template <int D, bool POOL, bool ONE, bool WIDE, bool TWO, int N>
__global__ void __launch_bounds__(kThreads) paged_kernel(PagedArgs<N> a) {
  static_assert(!POOL || D == kUnpack, "pool order is for stream-in");
  static_assert(!(ONE && WIDE), "wide launches look every unit up");
  static_assert(!TWO || (POOL && !ONE), "a wave's two blocks are looked up in pool order");
  const int lane = lane_id();
  const uint32_t ub = a.ub, heads = a.heads;
  // Tiles within one block keep the hardware's round-robin dealing in table
  // order: pool blocks are scattered by the block table anyway, and on MI355X
  // every XCD-grouped order measured was slower (by 2-8 %).  Pool order, and
  // table order with tiles across blocks, deal chunks of tiles.
  int64_t y = blockIdx.y;
  uint32_t tile = blockIdx.x;
  Seq q = {};
  int first_blk = 0;  // of the sequence's logical blocks
  int t0_l = 0, p_l = 0, p1_l = 0;
  if constexpr (POOL) {
    if constexpr (N == 64) {  // one sequence per lane, fetched beside the owner entry
      t0_l = a.s.t0[lane];
      p_l = a.s.tok[lane];
      p1_l = a.s.tok[lane + 1];
    }
    if constexpr (WIDE) {
      const uint64_t t = xcd_chunk<uint64_t>(tile + (uint64_t)y * a.tiles,
                                             (uint64_t)a.tiles * gridDim.y, kPoolChunk);
      y = (int64_t)(t / (uint32_t)a.tiles);
      tile = (uint32_t)(t - (uint64_t)y * a.tiles);
    } else {
      const uint32_t t = xcd_chunk<uint32_t>(tile + (uint32_t)y * a.tiles, a.tiles * gridDim.y,
                                             kPoolChunk);
      y = a.d_tiles.div(t);
      tile = t - (uint32_t)y * a.tiles;
    }
  } else {
    if constexpr (!ONE && !WIDE) {
      const uint32_t t = xcd_chunk<uint32_t>(tile + (uint32_t)y * a.tiles, a.tiles * gridDim.y,
                                             kTableChunk);
      y = a.d_tiles.div(t);
      tile = t - (uint32_t)y * a.tiles;
    }
    q = find_seq(a.s, tile);
    tile = q.k;
    first_blk = a.d_bs.div(q.t0);
  }
  u32x4* pool = (u32x4*)a.pool + (a.m.slab0 + y) * a.s_slab;
  u32x4* wire = (u32x4*)a.wire + y * a.m.w_slab;

  for (int step = 0; step < (WIDE ? a.steps : 1); ++step) {
    // The tile's first unit: unit r0 of head h0 of block j0.
    uint64_t f;
    uint32_t j0, h0, r0;
    if constexpr (WIDE) {
      f = ((uint64_t)tile * a.steps + step) * kPagedTile;
      const uint64_t hb = f / ub;
      r0 = (uint32_t)(f - hb * ub);
      j0 = (uint32_t)(hb / heads);
      h0 = (uint32_t)(hb - (uint64_t)j0 * heads);
    } else {
      f = tile * kPagedTile;
      const uint32_t hb = a.d_ub.div((uint32_t)f);
      r0 = (uint32_t)f - hb * ub;
      j0 = a.d_heads.div(hb);
      h0 = hb - j0 * heads;
    }
    Seq u = q;  // ONE: the block's sequence
    int blk1 = 0, j1 = 0;
    if constexpr (ONE && POOL) {
      blk1 = j0;
      const int own = __builtin_amdgcn_readfirstlane(a.owner[blk1]);
      if (own < 0) return;  // block not written by this call
      u.b = a.d_max.div(own);
      if (u.b >= a.nseq) return;
      j1 = own - u.b * a.max_blocks;
      if constexpr (N == 64) {
        u.t0 = __builtin_amdgcn_readlane(t0_l, u.b);
        u.p = __builtin_amdgcn_readlane(p_l, u.b);
        u.n = __builtin_amdgcn_readlane(p1_l, u.b) - u.p;
      } else {
        u.t0 = a.s.t0[u.b];
        u.p = a.s.tok[u.b];
        u.n = a.s.tok[u.b + 1] - u.p;
      }
    } else if constexpr (ONE) {
      j1 = first_blk + j0;
      blk1 = __builtin_amdgcn_readfirstlane(a.bt[(int64_t)u.b * a.max_blocks + j1]);
      if (blk1 < 0 || blk1 >= a.num_blocks) return;  // unmapped block: skipped
    }

    // TWO: a wave's units follow each other, so they lie in two blocks at most.
    // Both are looked up once for the wave and a lane takes one.
    uint32_t off0 = 0;  // the wave's first unit in its block
    Seq two[TWO ? 2 : 1] = {};  // k: the logical block; n: 0 where there is none
    if constexpr (TWO) {
      const uint32_t w0 = __builtin_amdgcn_readfirstlane(r0 + (threadIdx.x & ~63u) * kPagedUnroll);
      const uint32_t d = a.d_ub.div(w0), dj = a.d_heads.div(h0 + d);
      off0 = (h0 + d - dj * heads) * ub + (w0 - d * ub);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const uint32_t blk = j0 + dj + i, last = a.num_blocks - 1;
        const int own = __builtin_amdgcn_readfirstlane(a.owner[min(blk, last)]);
        const int b = a.d_max.div(max(own, 0));
        if (blk > last || own < 0 || b >= a.nseq) continue;
        two[i] = {b, own - b * a.max_blocks, a.s.t0[b], a.s.tok[b + 1] - a.s.tok[b], a.s.tok[b]};
      }
    }

    // Lanes whose unit lies outside the range (the first and last block of a
    // sequence, unmapped blocks) move nothing.
    int64_t po[kPagedUnroll], wo[kPagedUnroll];
    bool ok[kPagedUnroll];
#pragma unroll
    for (int i = 0; i < kPagedUnroll; ++i) {
      // On the way in a wave's units follow each other (2 KB written in order:
      // 1801 us against 1835 with the waves' units interleaved, LLaMA-2-70B pool
      // in pool order; 1964 against 1981 in table order); on the way out they
      // interleave (1 % faster).
      const uint32_t idx = D == kUnpack ? (threadIdx.x & ~63u) * kPagedUnroll + i * 64 + lane
                                        : i * kThreads + threadIdx.x;
      const bool second = TWO && off0 + i * 64 + lane >= (uint32_t)a.s_blk;
      const uint32_t z = TWO ? off0 + i * 64 + lane - (second ? (uint32_t)a.s_blk : 0) : r0 + idx;
      const uint32_t d = a.d_ub.div(z);
      const uint32_t e = z - d * ub;
      uint32_t h = h0 + d;
      Seq s = u;
      int j = j1;
      ok[i] = true;
      if constexpr (TWO) {
        h = d;
        s = two[second];
        j = s.k;
        po[i] = (int64_t)(f + idx);
      } else if constexpr (ONE) {
        po[i] = (int64_t)blk1 * a.s_blk + (int64_t)h0 * ub + r0 + idx;
      } else {
        const uint32_t dj = a.d_heads.div(h);
        h -= dj * heads;
        if constexpr (POOL) {
          const int blk = j0 + dj;
          ok[i] = blk < a.num_blocks;
          const int own = a.owner[min(blk, a.num_blocks - 1)];
          s.b = a.d_max.div(max(own, 0));
          ok[i] = ok[i] && own >= 0 && s.b < a.nseq;
          j = own - s.b * a.max_blocks;
          if (!ok[i]) s.b = 0;
          if constexpr (N == 64) {
            s.t0 = __shfl(t0_l, s.b, 64);
            s.p = __shfl(p_l, s.b, 64);
            s.n = __shfl(p1_l, s.b, 64) - s.p;
          } else {
            s.t0 = a.s.t0[s.b];
            s.p = a.s.tok[s.b];
            s.n = a.s.tok[s.b + 1] - s.p;
          }
          po[i] = (int64_t)(f + idx);
        } else {
          j = first_blk + j0 + dj;
          // past the sequence's last block the range test below fails
          const int blk = a.bt[(int64_t)s.b * a.max_blocks + min(j, a.max_blocks - 1)];
          ok[i] = blk >= 0 && blk < a.num_blocks;  // unmapped block: skipped
          po[i] = (int64_t)blk * a.s_blk + (int64_t)h * ub + e;
        }
      }
      // The unit's place in the head's run.  The last logical block ends below
      // 2^30 units and a tile reaches at most one tile past it, so nothing
      // here wraps.
      const int pu = j * (int)ub + (int)e - s.t0 * a.du;
      const int run = s.n * a.du;
      ok[i] = ok[i] && (uint32_t)pu < (uint32_t)run;
      wo[i] = (int64_t)s.p * ((int64_t)heads * a.du) + (int64_t)h * run + pu;
    }
    if constexpr (ONE) {
      // One access in flight per wave: load, store, and the store's end before
      // the next load.  With the chip full of waves that is enough, and random
      // blocks are served better: gather and pool-order scatter of the
      // LLaMA-2-70B pool, replayed, 1784 and 1759 us; without the last wait 1839
      // and 1780, with two loads in flight 1870 and 1850.
#pragma unroll
      for (int i = 0; i < kPagedUnroll; ++i) {
        if (ok[i])
          st_nt(ld_nt((D == kPack) ? pool + po[i] : wire + wo[i]),
                (D == kPack) ? wire + wo[i] : pool + po[i]);
        if (i + 1 < kPagedUnroll) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      }
    } else {
      // Both loads in flight (up to 2 % faster than one here, where a wave has
      // more to work out first), without guards: an idle lane reads the slab's
      // first unit instead.
      u32x4 v[kPagedUnroll];
#pragma unroll
      for (int i = 0; i < kPagedUnroll; ++i)
        v[i] = (D == kPack) ? ld_nt(pool + (ok[i] ? po[i] : 0))
                            : ld_nt(wire + (ok[i] ? wo[i] : 0));
#pragma unroll
      for (int i = 0; i < kPagedUnroll; ++i)
        if (ok[i]) st_nt(v[i], (D == kPack) ? wire + wo[i] : pool + po[i]);
    }
  }
}

// Owner map in one launch (see OwnerMapArgs).  Four chunks of a wave are in
// flight at a time: the launch is bound by their latency.
template <int N>
__global__ void __launch_bounds__(kOwnerThreads) owner_map_kernel(OwnerMapArgs<N> a) {
  __shared__ int s_own[kOwnerSpan];
  const int lane = lane_id();
  const int lo = blockIdx.x * kOwnerSpan;
  const int span = min(kOwnerSpan, a.num_blocks - lo);
  for (int i = threadIdx.x; i < span; i += kOwnerThreads) s_own[i] = -1;
  __syncthreads();
  constexpr int kWaves = kOwnerThreads / 64, kDeep = 4;
  for (int c0 = threadIdx.x >> 6; c0 < a.chunks; c0 += kWaves * kDeep) {
    int entry[kDeep], blk[kDeep];
#pragma unroll
    for (int i = 0; i < kDeep; ++i) {
      const int c = min(c0 + i * kWaves, a.chunks - 1);  // past the end: the last one again
      const Seq q = find_seq(a.s, c);
      const int last = a.d_bs.div(q.t0 + q.n - 1);
      entry[i] = q.b * a.max_blocks + min((int)a.d_bs.div(q.t0) + q.k * 64 + lane, last);
      blk[i] = a.bt[entry[i]];
    }
#pragma unroll
    for (int i = 0; i < kDeep; ++i)
      if (blk[i] >= lo && blk[i] < lo + span) s_own[blk[i] - lo] = entry[i];
  }
  __syncthreads();
  for (int i = threadIdx.x; i < span; i += kOwnerThreads) a.owner[lo + i] = s_own[i];
}

// Owner map (see OwnerArgs): a clearing pass, then one lane per table entry.
__global__ void __launch_bounds__(kThreads) owner_clear_kernel(OwnerArgs a) {
  const int i = blockIdx.x * kThreads + threadIdx.x;
  if (i < a.num_blocks) a.owner[i] = -1;
}

__global__ void __launch_bounds__(kThreads) claims_clear_kernel(OwnerArgs a) {
  const int i = blockIdx.x * kThreads + threadIdx.x;
  if (i < a.num_blocks) a.owner[i] = 0;
}

// One lane per table entry, as owner_build_kernel; counts instead of storing.
__global__ void __launch_bounds__(kThreads) claims_count_kernel(OwnerArgs a) {
  const int b = blockIdx.y;
  const int j = blockIdx.x * kThreads + threadIdx.x;
  if (j >= a.max_blocks) return;
  const int t0 = a.r.t0[b], t1 = t0 + a.r.n[b];
  if (t0 >= t1 || (j + 1) * a.block_size <= t0 || j * a.block_size >= t1) return;
  const int blk = a.bt[(int64_t)(a.b0 + b) * a.max_blocks + j];
  if (blk < 0 || blk >= a.num_blocks) return;
  atomicAdd(&a.owner[blk], 1);
}

__global__ void __launch_bounds__(kThreads) owner_build_kernel(OwnerArgs a) {
  const int b = blockIdx.y;
  const int j = blockIdx.x * kThreads + threadIdx.x;
  if (j >= a.max_blocks) return;
  const int t0 = a.r.t0[b], t1 = t0 + a.r.n[b];
  if (t0 >= t1 || (j + 1) * a.block_size <= t0 || j * a.block_size >= t1) return;
  const int gb = a.b0 + b;  // the sequence's index in the call
  const int blk = a.bt[(int64_t)gb * a.max_blocks + j];
  if (blk < 0 || blk >= a.num_blocks) return;
  a.owner[blk] = gb * a.max_blocks + j;
}

// Finds rows [row0, row0 + rows) of a launch's slab, one per lane, shared out by
// waves: store(row - row0, sequence, head, token) leaves them in LDS.  The
// caller synchronises.
template <int N, bool SEARCH, typename Args, typename F>
__device__ __forceinline__ void find_rows(const Args& a, uint32_t row0, uint32_t rows, F store) {
  const int lane = lane_id();
  // Every lane of a wave that has rows takes one (the last one again past the
  // end), so that lanes can read each other's sequences.
  for (uint32_t k = threadIdx.x & ~63u; k < rows; k += kThreads) {
    const uint32_t r = row0 + min(k + lane, rows - 1);
    const uint32_t q = a.d_heads.div(r);  // tok[b] <= q < tok[b + 1]
    const int qlo = a.d_heads.div(row0 + k);
    const int qhi = a.d_heads.div(row0 + min(k + 63, rows - 1));
    int b, b1, p, t0, seq;
    if constexpr (N == 64) {
      const int tok = a.tok[lane];
      b = __popcll(__ballot(tok <= qlo)) - 1;
      b1 = __popcll(__ballot(tok <= qhi)) - 1;
      // The wave's rows lie in sequences [b, b1]: a step for each, or past eight
      // a search (27 sequences of 1-2 tokens, one head, 8 layers: 3.1 us by
      // steps, 2.4 by search; 6 sequences 2.0 and 2.1).  The split-key rows,
      // launches of 4 MB and more whose waves hold few, go without (one sequence
      // of 16 tokens, 44 heads, 10 MB: 4.8 us, 5.2 with the search compiled in).
      const int steps = b1 - b;
      if (!SEARCH || steps <= 8) {
        const int b0 = b;
        for (int i = b0 + 1; i <= b1; ++i) b += __builtin_amdgcn_readlane(tok, i) <= (int)q;
      } else {
        int hi = b1;
#pragma unroll
        for (int i = 0; i < 6; ++i) {  // 63 sequences past the first at most
          const int mid = (b + hi + 1) >> 1;
          const bool at = __shfl(tok, mid, 64) <= (int)q;
          b = at ? mid : b;
          hi = at ? hi : mid - 1;
        }
      }
      p = __shfl(tok, b, 64);
      t0 = __shfl(a.t0[lane], b, 64);
      seq = __shfl(a.seq[lane], b, 64);
    } else {
      b = b1 = -1;
#pragma unroll
      for (int i = 0; i < N / 64; ++i) {
        const int tok = a.tok[i * 64 + lane];
        b += __popcll(__ballot(tok <= qlo));
        b1 += __popcll(__ballot(tok <= qhi));
      }
      const int b0 = b;
      for (int i = b0 + 1; i <= b1; ++i) b += a.tok[i] <= (int)q;
      p = a.tok[b];
      t0 = a.t0[b];
      seq = a.seq[b];
    }
    const uint32_t n = a.tok[b + 1] - p, rr = r - (uint32_t)p * a.heads;
    const uint32_t h = rr / n;
    if (k + lane < rows) store(k + lane, seq, h, t0 + (rr - h * n));
  }
}

// ---------------------------------------------------------------------------
// Short runs: grid (ceil(total / (256 * U)), nslabs); see RowArgs.  Each lane
// moves U units of its slab, 256 apart.
//
// Small calls are bound by the launch and by one chain of dependent loads
// (arguments, the sequence's place, a table entry, the data), larger ones by
// instructions: what a unit costs to find.  Where every sequence has the same
// number of tokens (a decode step), three multiplications find it.  Ragged
// rows are found once per row, by as many lanes as the workgroup has rows, and
// left in LDS for the units.  Before, every unit searched for its sequence and
// divided three times, 64 sequences to a launch and a split-key cache's halves
// apart (graph replays, one way in and one out): 32 sequences of 1-8 tokens, 8
// heads x 128 x 2 bytes, 20 layers, paged, 16.3 -> 11.2 us; one token of 256
// such sequences 36.6 -> 20.0; of 8 sequences of 72 heads, 16 layers, split
// key, 19.7 -> 15.0; of 8 sequences of 40 heads, 10 layers, dense, 4.9 -> 4.3.
// ---------------------------------------------------------------------------
template <int D, int U, bool EVEN, int N>
__global__ void __launch_bounds__(kThreads) rows_kernel(RowArgs<N> a) {
  const int64_t y = blockIdx.y;
  const int half = (int)(y & 1);  // the launch starts at a layer's key slab
  u32x4* cache = (u32x4*)a.cache + (a.m.slab0 + y) * a.s_slab;
  u32x4* wire = (u32x4*)a.wire + y * a.m.w_slab;
  const int64_t s_tok = a.s_tok[half], s_e = a.s_e[half];
  const uint32_t first = blockIdx.x * (kThreads * U);
  const uint32_t last = min(first + kThreads * U, (uint32_t)a.total) - 1;

  // Cache offset of token s of head h of the sequence; negative where its block
  // is unmapped (skipped).
  auto row_offset = [&](int seq, uint32_t h, uint32_t s) -> int64_t {
    int64_t o = (int64_t)h * a.s_h;
    if (!a.paged) return o + (int64_t)seq * a.s_b + (int64_t)s * s_tok;
    const uint32_t j = a.d_bs.div(s);
    const int blk = a.bt[(int64_t)seq * a.max_blocks + j];
    if (blk < 0 || blk >= a.num_blocks) return -1;
    return o + (int64_t)blk * a.s_b + (int64_t)(s - j * a.block_size) * s_tok;
  };

  __shared__ int64_t s_off[EVEN ? 1 : kThreads * U + 1];
  const uint32_t row0 = EVEN ? 0 : a.d_du.div(first);
  if constexpr (!EVEN) {
    const uint32_t rows = a.d_du.div(last) - row0 + 1;
    find_rows<N, true>(a, row0, rows, [&](uint32_t i, int seq, uint32_t h, uint32_t s) {
      s_off[i] = row_offset(seq, h, s);
    });
    __syncthreads();
  }

  // Loads carry no guard (a lane past the end reads the last unit again, one
  // of an unmapped block the slab's first), so they issue back to back.
  int64_t co[U];
  u32x4 v[U];
#pragma unroll
  for (int i = 0; i < U; ++i) {
    const uint32_t u = min(first + i * kThreads + threadIdx.x, last);
    const uint32_t row = a.d_du.div(u);
    const uint32_t g = u - row * a.du;
    if constexpr (EVEN) {
      const uint32_t b = a.d_seq.div(row);
      const uint32_t rr = row - b * (uint32_t)(a.heads * a.n);
      const uint32_t h = a.d_n.div(rr);
      co[i] = row_offset(a.seq[b], h, a.t0[b] + (rr - h * a.n));
    } else {
      co[i] = s_off[row - row0];
    }
    if (co[i] >= 0) co[i] += (int64_t)g * s_e;
    v[i] = (D == kPack) ? ld_nt(cache + (co[i] >= 0 ? co[i] : 0)) : ld_nt(wire + u);
  }
#pragma unroll
  for (int i = 0; i < U; ++i) {
    const uint32_t u = first + i * kThreads + threadIdx.x;
    if (u <= last && co[i] >= 0) st_nt(v[i], (D == kPack) ? wire + u : cache + co[i]);
  }
}

// ---------------------------------------------------------------------------
// Short runs of two tokens and more in a split-key cache: grid (ceil(rows /
// a.tile), nslabs); a workgroup takes a.tile rows of its slab.  The tokens of a
// run stand side by side in each group of the key half, so a key slab's tile
// is moved with lanes along the rows on the cache side and through LDS: a
// lane per wire unit would touch each 128-byte line once per token (43 layers,
// 29 heads x 256 x 2 bytes, 3 sequences of 1-3 tokens: 7.1 and 13.5 us out and
// in that way, 6.3 and 10.2 this way).
// ---------------------------------------------------------------------------
template <int D, int N>
__global__ void __launch_bounds__(kThreads) split_rows_kernel(RowArgs<N> a) {
  extern __shared__ u32x4 lds[];  // a.tile rows of du + 1 units, then their offsets
  const int64_t y = blockIdx.y;
  const int half = (int)(y & 1);
  u32x4* cache = (u32x4*)a.cache + (a.m.slab0 + y) * a.s_slab;
  u32x4* wire = (u32x4*)a.wire + y * a.m.w_slab;
  const uint32_t du = a.du, pitch = du + 1;
  const int64_t s_tok = a.s_tok[half], s_e = a.s_e[half];
  int64_t* s_off = (int64_t*)(lds + a.tile * pitch);
  const uint32_t row0 = blockIdx.x * a.tile;
  const uint32_t rows = min((uint32_t)a.tile, a.d_du.div(a.total) - row0);
  find_rows<N, false>(a, row0, rows, [&](uint32_t i, int seq, uint32_t h, uint32_t s) {
    s_off[i] = (int64_t)seq * a.s_b + (int64_t)h * a.s_h + (int64_t)s * s_tok;
  });
  __syncthreads();
  wire += (int64_t)row0 * du;
  const uint32_t units = rows * du;
  u32x4 v[kRowsUnroll];
  int64_t co[kRowsUnroll];
  u32x4* at[kRowsUnroll];  // the unit's place in LDS, cache side
#pragma unroll
  for (int i = 0; i < kRowsUnroll; ++i) {
    const uint32_t j = min(i * kThreads + threadIdx.x, units - 1);
    uint32_t r, g;
    if (half) {  // value slab: units in wire order on both sides
      r = a.d_du.div(j);
      g = j - r * du;
    } else {     // key slab: rows fastest
      g = rows == (uint32_t)a.tile ? a.d_tile.div(j) : j / rows;
      r = j - g * rows;
    }
    co[i] = s_off[r] + (int64_t)g * s_e;
    at[i] = lds + r * pitch + g;
    v[i] = (D == kPack) ? ld_nt(cache + co[i]) : ld_nt(wire + j);
  }
  if (half) {
#pragma unroll
    for (int i = 0; i < kRowsUnroll; ++i) {
      const uint32_t j = i * kThreads + threadIdx.x;
      if (j < units) st_nt(v[i], (D == kPack) ? wire + j : cache + co[i]);
    }
    return;
  }
  // Place of wire unit j (group j % du of row j / du) in LDS.
  auto wire_at = [&](uint32_t j) { return lds + j + a.d_du.div(j); };
#pragma unroll
  for (int i = 0; i < kRowsUnroll; ++i) {
    const uint32_t j = i * kThreads + threadIdx.x;
    if (j < units) *((D == kPack) ? at[i] : wire_at(j)) = v[i];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kRowsUnroll; ++i) {
    const uint32_t j = i * kThreads + threadIdx.x;
    if (j < units) st_nt((D == kPack) ? *wire_at(j) : *at[i], (D == kPack) ? wire + j : cache + co[i]);
  }
}

// ---------------------------------------------------------------------------
// Split-key caches: grid (tiles_per_slab, nslabs); a tile is a.tile tokens of
// one (sequence, head).  A key slab holds the head as [group][token] (each
// group 16 bytes), the wire as [token][group]: the tile is read with lanes
// along the contiguous axis of the source, transposed through LDS (rows of du
// + 1 units: the padding unit keeps column accesses on distinct banks), and
// written with lanes along the contiguous axis of the destination.  A value
// slab's tile is contiguous on both sides.
//
// Bound by HBM for whole prompts: the OPT-13B stage's split-key shape (1.28 GB)
// takes 397 and 396 us one way, 6.3 TB/s, against 402 and 399 in two launches
// with key tiles of 16 KB (4 workgroups to a CU); small prompts gain the launch
// (10 layers, one head, 254 tokens: 5.7 -> 2.5 us).  Tiles that end inside lines
// write those twice, each time in part: 16 sequences of 300-1100 tokens at
// positions 0-200, 20 heads, 32 groups a token, 399 MB, 138.2 and 158.9 us out and
// in, 132.1 and 132.3 with tiles that end on lines; 16 groups, 331 MB, 112.2 and
// 118.7, 110.1 and 110.0.
// ---------------------------------------------------------------------------
template <int D, int U, int N>
__global__ void __launch_bounds__(kThreads) split_kernel(SplitArgs<N> a) {
  extern __shared__ u32x4 lds[];
  uint32_t tile, y;
  xcd_tile(a.deal, &tile, &y);
  const Seq q = find_seq(a.s, tile);
  const uint32_t lead = (a.line0 + q.t0) & a.line_mask;
  const uint32_t tpr = a.d_tile.div(lead + q.n + a.tile - 1);  // tiles per run
  const uint32_t h = (uint32_t)q.k / tpr, k = (uint32_t)q.k - h * tpr;
  const uint32_t du = a.du, tok0 = k ? k * a.tile - lead : 0;
  const uint32_t ntk = min((k + 1) * a.tile - lead, (uint32_t)q.n) - tok0;
  const uint32_t units = ntk * du;
  u32x4* head = (u32x4*)a.cache + (int64_t)(a.m.slab0 + y) * a.s_slab + (int64_t)(a.b0 + q.b) * a.s_b +
                (int64_t)h * a.s_h;
  u32x4* wire = (u32x4*)a.wire + (int64_t)y * a.m.w_slab +
                (int64_t)q.p * ((int64_t)a.heads * du) + ((int64_t)h * q.n + tok0) * du;
  u32x4 v[U];
  if (y & 1) {  // value slab
    u32x4* run = head + (int64_t)(q.t0 + tok0) * du;
    const u32x4* src = (D == kPack) ? run : wire;
    u32x4* dst = (D == kPack) ? wire : run;
#pragma unroll
    for (int i = 0; i < U; ++i)
      v[i] = ld_nt(src + min(i * kThreads + threadIdx.x, units - 1));
#pragma unroll
    for (int i = 0; i < U; ++i) {
      const uint32_t idx = i * kThreads + threadIdx.x;
      if (idx < units) st_nt(v[i], dst + idx);
    }
    return;
  }
  // Key slab: unit j of the cache side is token j % a.tile of group j / a.tile,
  // unit j of the wire side group j % du of token j / du.
  u32x4* key = head + q.t0 + tok0;
  const int64_t S = a.seq_cap;
  const uint32_t pitch = du + 1;
  uint32_t g[U], t[U];
#pragma unroll
  for (int i = 0; i < U; ++i) {
    const uint32_t j = i * kThreads + threadIdx.x;
    g[i] = a.d_tile.div(j);
    t[i] = j - g[i] * a.tile;
  }
#pragma unroll
  for (int i = 0; i < U; ++i) {
    const uint32_t j = min(i * kThreads + threadIdx.x, units - 1);
    v[i] = (D == kPack) ? ld_nt(key + min(g[i], du - 1) * S + min(t[i], ntk - 1)) : ld_nt(wire + j);
  }
  if constexpr (D == kPack) {
#pragma unroll
    for (int i = 0; i < U; ++i)
      if (g[i] < du && t[i] < ntk) lds[t[i] * pitch + g[i]] = v[i];
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < U; ++i) {
    const uint32_t j = i * kThreads + threadIdx.x;
    if (j < units) {
      const uint32_t wt = a.d_du.div(j);
      u32x4* at = lds + wt * pitch + (j - wt * du);
      if (D == kPack) st_nt(*at, wire + j);
      else *at = v[i];
    }
  }
  if constexpr (D == kUnpack) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < U; ++i)
      if (g[i] < du && t[i] < ntk) st_nt(lds[t[i] * pitch + g[i]], key + g[i] * S + t[i]);
  }
}

// ---------------------------------------------------------------------------
// Cache-to-cache copy: grid (ceil(total / (256 * kCopyUnroll)), nslabs).  The
// units of a slab's ranges in wire order, as in the short-run kernel, but
// straight from the source cache to the same logical place in the destination
// cache.  Used for swaps whose rows are too narrow for DMA to run efficiently (a
// decode step's one-token update is 256-byte rows); on pinned host memory each
// lane's store or load crosses the host link.
//
// Bound by the link's requests of narrow rows: 4.72 MB in 18432 rows of 256
// bytes take 90 us out and 113 us in, where a contiguous copy takes 83.  The
// stores are ordinary ones: nontemporal, they took 98 us out.  One unit per
// lane: with two, 132 MB of 7-31 KB rows came in in 2.44 ms instead of 2.41.
// Up to 256 sequences go in a launch: 171 of one token, 0.44 MB, 12.8 us out
// and 25 in, in three launches 20 and 34.
// ---------------------------------------------------------------------------
template <int N>
__global__ void __launch_bounds__(kThreads) copy_kernel(CopyArgs<N> a) {
  constexpr int U = kCopyUnroll;
  __shared__ int64_t s_src[kThreads * U], s_dst[kThreads * U];
  const uint32_t first = blockIdx.x * (kThreads * U);
  const uint32_t last = min(first + kThreads * U, (uint32_t)a.total) - 1;
  const uint32_t row0 = a.d_du.div(first);
  find_rows<N, true>(a, row0, a.d_du.div(last) - row0 + 1,
                     [&](uint32_t i, int seq, uint32_t h, uint32_t s) {
                       const int64_t e = (int64_t)s * a.du;
                       s_src[i] = (int64_t)seq * a.s_b + (int64_t)h * a.s_h + e;
                       s_dst[i] = (int64_t)seq * a.d_b + (int64_t)h * a.d_h + e;
                     });
  __syncthreads();
  const int64_t slab = a.slab0 + (int64_t)blockIdx.y;
  const u32x4* src = (const u32x4*)a.src + slab * a.s_slab;
  u32x4* dst = (u32x4*)a.dst + slab * a.d_slab;
  u32x4 v[U];
  int64_t to[U];
#pragma unroll
  for (int i = 0; i < U; ++i) {
    const uint32_t u = min(first + i * kThreads + threadIdx.x, last);
    const uint32_t row = a.d_du.div(u), g = u - row * a.du;
    to[i] = s_dst[row - row0] + g;
    v[i] = ld_nt(src + s_src[row - row0] + g);
  }
#pragma unroll
  for (int i = 0; i < U; ++i)
    if (first + i * kThreads + threadIdx.x <= last) dst[to[i]] = v[i];
}

}  // namespace

namespace {

// Launch with the runtime's own status for this launch (a stale error left by
// an unrelated earlier call is not picked up, unlike hipGetLastError).  A grid too
// wide for one is refused here as the runtime would refuse it.
template <typename Args>
hipError_t launch(const void* fn, dim3 grid, const Args& a, hipStream_t s, size_t lds = 0) {
  if (grid.x == 0 || grid.y == 0) return hipSuccess;
  if (grid.x >= kMaxGroups) return hipErrorInvalidConfiguration;
  void* args[] = {const_cast<Args*>(&a)};
  return hipLaunchKernel(fn, grid, dim3(kThreads), args, lds, s);
}

}  // namespace

template <int N>
hipError_t launch_dense_runs(int dir, const DenseRunArgs<N>& a, uint32_t nslabs, hipStream_t s) {
  const void* fn = dir == kPack ? (const void*)&dense_runs_kernel<kPack, N>
                                : (const void*)&dense_runs_kernel<kUnpack, N>;
  return launch(fn, dim3(a.deal.tiles, nslabs), a, s);
}
template hipError_t launch_dense_runs<kSeqPerLaunch>(int, const DenseRunArgs<kSeqPerLaunch>&,
                                                     uint32_t, hipStream_t);
template hipError_t launch_dense_runs<kSeqMany>(int, const DenseRunArgs<kSeqMany>&, uint32_t,
                                                hipStream_t);

namespace {

template <int N, bool ONE, bool WIDE>
const void* paged_fn(int dir, bool pool, bool two) {
  if constexpr (!ONE && N != kSeqPerLaunch)
    if (pool && two) return (const void*)&paged_kernel<kUnpack, true, false, WIDE, true, N>;
  if (pool) return (const void*)&paged_kernel<kUnpack, true, ONE, WIDE, false, N>;
  return dir == kPack ? (const void*)&paged_kernel<kPack, false, ONE, WIDE, false, N>
                      : (const void*)&paged_kernel<kUnpack, false, ONE, WIDE, false, N>;
}

}  // namespace

template <int N>
hipError_t launch_paged(int dir, const PagedArgs<N>& a, bool wide, uint32_t nslabs,
                        hipStream_t s) {
  const bool pool = a.owner != nullptr;
  // Pool order, more than 64 sequences, tiles across blocks: a look-up per lane
  // ends in three loads of its own from the arguments.  Look-ups by lane and by
  // wave: 193 sequences, blocks of 1792 units, three fifths of the pool, 430 MB,
  // 168.6 and 150.2 us; 100 of 128 units, 2.09 GB, 750 and 696; 80 of 1280 units,
  // the whole pool, 2.23 GB, 729 and 737.  (Up to 64 the ranges are in the lanes:
  // 526 and 548 with the whole pool written, 342 and 333 with three fifths.)
  // Smaller blocks are more than two to a wave, larger ones past 32 bits.
  const bool two = a.s_blk >= 64 * kPagedUnroll && a.s_blk <= (1 << 30);
  const void* fn = wide                          ? paged_fn<N, false, true>(dir, pool, two)
                   : a.s_blk % kPagedTile == 0 ? paged_fn<N, true, false>(dir, pool, two)
                                               : paged_fn<N, false, false>(dir, pool, two);
  return launch(fn, dim3(a.tiles, nslabs), a, s);
}
template hipError_t launch_paged<kSeqPerLaunch>(int, const PagedArgs<kSeqPerLaunch>&, bool,
                                                uint32_t, hipStream_t);
template hipError_t launch_paged<kSeqMany>(int, const PagedArgs<kSeqMany>&, bool, uint32_t,
                                           hipStream_t);
// Workgroups of kThreads lanes covering n items (n up to INT32_MAX).
static uint32_t groups_of(int32_t n) { return (uint32_t)(((int64_t)n + kThreads - 1) / kThreads); }

hipError_t launch_owner_clear(const OwnerArgs& a, hipStream_t s) {
  return launch((const void*)&owner_clear_kernel, dim3(groups_of(a.num_blocks)), a, s);
}

hipError_t launch_owner_build(const OwnerArgs& a, hipStream_t s) {
  return launch((const void*)&owner_build_kernel, dim3(groups_of(a.max_blocks), a.nseq), a, s);
}

template <int N>
hipError_t launch_owner_map(const OwnerMapArgs<N>& a, hipStream_t s) {
  void* args[] = {const_cast<OwnerMapArgs<N>*>(&a)};
  const uint32_t groups = (uint32_t)(((int64_t)a.num_blocks + kOwnerSpan - 1) / kOwnerSpan);
  return hipLaunchKernel((const void*)&owner_map_kernel<N>, dim3(groups), dim3(kOwnerThreads),
                         args, 0, s);
}
template hipError_t launch_owner_map<kSeqPerLaunch>(const OwnerMapArgs<kSeqPerLaunch>&,
                                                    hipStream_t);
template hipError_t launch_owner_map<kSeqMany>(const OwnerMapArgs<kSeqMany>&, hipStream_t);

hipError_t launch_block_claims(const OwnerArgs& a, bool clear, hipStream_t s) {
  if (clear) {
    const hipError_t e =
        launch((const void*)&claims_clear_kernel, dim3(groups_of(a.num_blocks)), a, s);
    if (e != hipSuccess) return e;
  }
  return launch((const void*)&claims_count_kernel, dim3(groups_of(a.max_blocks), a.nseq), a, s);
}

template <int N>
hipError_t launch_rows(int dir, bool even, const RowArgs<N>& a, uint32_t nslabs, hipStream_t s) {
  // Even launches take one unit per lane at every size (paged step of 256
  // sequences, 10.5 MB: 9.8 us one way against 10.4 with two; 82 MB: 31.0
  // against 32.0); ragged ones two from 4 MB on, where a workgroup's rows and
  // barrier count (5.9 MB: 5.6 against 6.6 us; 144 MB: 50 against 55).
  const bool two = !even && (uint64_t)a.total * nslabs >= (1ull << 18);
  const uint32_t per = kThreads * (two ? 2 : 1);
  const void* fn;
  if (dir == kPack)
    fn = even  ? (const void*)&rows_kernel<kPack, 1, true, N>
         : two ? (const void*)&rows_kernel<kPack, 2, false, N>
               : (const void*)&rows_kernel<kPack, 1, false, N>;
  else
    fn = even  ? (const void*)&rows_kernel<kUnpack, 1, true, N>
         : two ? (const void*)&rows_kernel<kUnpack, 2, false, N>
               : (const void*)&rows_kernel<kUnpack, 1, false, N>;
  return launch(fn, dim3((uint32_t)(((uint64_t)a.total + per - 1) / per), nslabs), a, s);
}
template <int N>
hipError_t launch_split_rows(int dir, const RowArgs<N>& a, uint32_t nslabs, hipStream_t s) {
  const void* fn = dir == kPack ? (const void*)&split_rows_kernel<kPack, N>
                                : (const void*)&split_rows_kernel<kUnpack, N>;
  const uint32_t rows = (uint32_t)(a.total / a.du);
  const size_t lds = (size_t)a.tile * ((a.du + 1) * 16 + 8);
  return launch(fn, dim3((rows + a.tile - 1) / a.tile, nslabs), a, s, lds);
}
template hipError_t launch_split_rows<kSeqPerLaunch>(int, const RowArgs<kSeqPerLaunch>&, uint32_t,
                                                     hipStream_t);
template hipError_t launch_split_rows<kSeqMany>(int, const RowArgs<kSeqMany>&, uint32_t,
                                                hipStream_t);
template hipError_t launch_rows<kSeqPerLaunch>(int, bool, const RowArgs<kSeqPerLaunch>&, uint32_t,
                                               hipStream_t);
template hipError_t launch_rows<kSeqMany>(int, bool, const RowArgs<kSeqMany>&, uint32_t,
                                          hipStream_t);

template <int N>
hipError_t launch_split(int dir, const SplitArgs<N>& a, uint32_t nslabs, hipStream_t s) {
  const int units = a.tile * a.du <= kThreads * 2 ? 2 : a.tile * a.du <= kThreads * 6 ? 6 : 8;
  const void* fn;
  if (dir == kPack)  // eight is for stream-in only
    fn = units == 2 ? (const void*)&split_kernel<kPack, 2, N>
                    : (const void*)&split_kernel<kPack, 6, N>;
  else
    fn = units == 2   ? (const void*)&split_kernel<kUnpack, 2, N>
         : units == 6 ? (const void*)&split_kernel<kUnpack, 6, N>
                      : (const void*)&split_kernel<kUnpack, 8, N>;
  // Six units per lane: at most 4 workgroups to a CU (259 and 269 us as above;
  // as many as fit 264 and 277); eight need nearly as much.
  const size_t lds = units > 2 ? kSplitLdsFor4 : (size_t)a.tile * (a.du + 1) * 16;
  return launch(fn, dim3(a.deal.tiles, nslabs), a, s, lds);
}
template hipError_t launch_split<kSeqPerLaunch>(int, const SplitArgs<kSeqPerLaunch>&, uint32_t,
                                                hipStream_t);
template hipError_t launch_split<kSeqMany>(int, const SplitArgs<kSeqMany>&, uint32_t,
                                           hipStream_t);

template <int N>
hipError_t launch_copy(const CopyArgs<N>& a, uint32_t nslabs, hipStream_t s) {
  const uint32_t per = kThreads * kCopyUnroll;
  return launch((const void*)&copy_kernel<N>,
                dim3((uint32_t)(((uint64_t)a.total + per - 1) / per), nslabs), a, s);
}
template hipError_t launch_copy<kSeqPerLaunch>(const CopyArgs<kSeqPerLaunch>&, uint32_t,
                                               hipStream_t);
template hipError_t launch_copy<kSeqMany>(const CopyArgs<kSeqMany>&, uint32_t, hipStream_t);

}  // namespace dv
