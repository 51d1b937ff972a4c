// C-ABI entry points: host-side validation, sizing and kernel/DMA dispatch.
// Everything is checked before the first enqueue, so an error return leaves
// the streams and all memory untouched.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <vector>

#include "../../include/dv.h"
#include "dv_host.h"
#include "dv_internal.h"

namespace {

using dv::kSeqPerLaunch;

// Swaps whose rows (one sequence's tokens of one head) are narrower than
// this go through the copy kernel instead of DMA.  Measured on MI355X for
// the OPT-66B stage: a one-token update (256-byte rows) took 162 us by one
// 2-D DMA and 2.5 ms by per-sequence DMA with ragged positions, against
// 90 to 113 us by kernel; rows of whole prompts move faster by DMA
// (57 GB/s against 54 GB/s), which leaves the compute units to other streams.
constexpr int64_t kNarrowRowBytes = 64 * 1024;

// Streams whose longest (sequence, head) run has at most this many 16-byte
// units use the short-run kernels; longer runs the tiled ones, except where
// they would leave many of a tile's lanes idle (run_stream).
constexpr int64_t kSmallRunUnits = 256;

// A validated view of one microbatch of a cache, sizes in 16-byte units.
struct View {
  int kind;
  int mem;
  int64_t L, H, D, B, E;
  int64_t du;        // units per token
  int64_t cap;       // token capacity per sequence
  int64_t S;         // dense kinds: max_seq
  int64_t bs, NB, max_blocks;
  char* base;
  const int32_t* bt;
  int32_t* owner;    // paged: optional owner-map workspace [NB]
  uint64_t bytes;    // storage bytes of the microbatch
};

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// The layout of a descriptor, without a microbatch (sizing calls).
int layout_of(const dv_cache* c, View* v) {
  if (!c || !c->mb_base) return DV_ERR_INVALID;
  if (c->elem_bytes <= 0 || c->num_layers <= 0 || c->num_heads <= 0 || c->head_dim <= 0 ||
      c->batch <= 0 || c->num_mb <= 0)
    return DV_ERR_INVALID;
  if (((int64_t)c->head_dim * c->elem_bytes) % 16 != 0) return DV_ERR_INVALID;
  if (c->mem != DV_MEM_DEVICE && c->mem != DV_MEM_HOST_PINNED) return DV_ERR_INVALID;
  v->kind = c->kind;
  v->mem = c->mem;
  v->L = c->num_layers;
  v->H = c->num_heads;
  v->D = c->head_dim;
  v->B = c->batch;
  v->E = c->elem_bytes;
  v->du = v->D * v->E / 16;
  v->S = v->bs = v->NB = v->max_blocks = 0;
  v->bt = nullptr;
  v->owner = nullptr;
  if (c->kind == DV_DENSE || c->kind == DV_DENSE_KSPLIT) {
    if (c->max_seq <= 0) return DV_ERR_INVALID;
    v->S = v->cap = c->max_seq;
    v->bytes = (uint64_t)v->L * 2 * v->B * v->H * v->S * v->du * 16;
  } else if (c->kind == DV_PAGED) {
    if (c->block_size <= 0 || c->num_blocks <= 0 || c->max_blocks <= 0 || !c->block_table)
      return DV_ERR_INVALID;
    v->bs = c->block_size;
    v->NB = c->num_blocks;
    v->max_blocks = c->max_blocks;
    v->cap = v->bs * v->max_blocks;
    v->bytes = (uint64_t)v->L * 2 * v->NB * v->H * v->bs * v->du * 16;
  } else {
    return DV_ERR_INVALID;
  }
  // Extents whose products the kernels take in 32-bit arithmetic (a launch's
  // first slab index, 2 * layer + 1, among them).
  if (v->L > (1 << 24) || v->cap > (1 << 24) || v->du > (1 << 16) || v->H * v->du > (1 << 20) ||
      v->cap * v->du > (1ll << 30))
    return DV_ERR_UNSUPPORTED;
  // A paged tile may reach past a sequence's last block, and a unit's place in
  // the head's run is counted from the sequence's first: capacity and one block
  // together must stay well inside int32.
  if (c->kind == DV_PAGED && v->bs * v->du > (1ll << 29)) return DV_ERR_UNSUPPORTED;
  // Every byte count derived from the descriptor stays far inside 64 bits:
  // its storage and the longest stream it can produce (all layers, every
  // sequence at full capacity) must be below 2^48 bytes.
  using u128 = unsigned __int128;
  const u128 per_token = (u128)v->L * 2 * v->H * v->du * 16;
  const u128 rows = c->kind == DV_PAGED ? (u128)v->NB * v->bs : (u128)v->B * v->S;
  const u128 limit = (u128)1 << 48;
  if (per_token * rows >= limit || per_token * v->B * v->cap >= limit) return DV_ERR_UNSUPPORTED;
  v->base = nullptr;
  return DV_OK;
}

// The layout plus microbatch mb's base address (and table, owner map).
int view_of(const dv_cache* c, int32_t mb, View* v) {
  const int rc = layout_of(c, v);
  if (rc != DV_OK) return rc;
  if (mb < 0 || mb >= c->num_mb) return DV_ERR_RANGE;
  v->base = static_cast<char*>(c->mb_base[mb]);
  if (!v->base || !aligned16(v->base)) return DV_ERR_INVALID;
  if (c->kind == DV_PAGED) {
    v->bt = c->block_table[mb];
    if (!v->bt) return DV_ERR_INVALID;
    v->owner = c->block_owner ? c->block_owner[mb] : nullptr;
    if ((reinterpret_cast<uintptr_t>(v->owner) & 3u) != 0) return DV_ERR_INVALID;
  }
  return DV_OK;
}

// Checks the ranges and returns the per-sequence (t0, n) and N.
int ranges_of(const View& v, int32_t l0, int32_t l1, const int32_t* t0, const int32_t* t1,
              std::vector<int32_t>* r0, std::vector<int32_t>* rn, int64_t* N) {
  if (!t1) return DV_ERR_INVALID;
  if (l0 < 0 || l1 < l0 || l1 > v.L) return DV_ERR_RANGE;
  r0->resize(v.B);
  rn->resize(v.B);
  int64_t total = 0;
  for (int64_t b = 0; b < v.B; ++b) {
    const int64_t a = t0 ? t0[b] : 0, e = t1[b];
    if (a < 0 || e < a || e > v.cap) return DV_ERR_RANGE;
    (*r0)[b] = (int32_t)a;
    (*rn)[b] = (int32_t)(e - a);
    total += e - a;
  }
  *N = total;
  return DV_OK;
}

uint64_t wire_bytes(const View& v, int32_t l0, int32_t l1, int64_t N) {
  return (uint64_t)(l1 - l0) * 2 * v.H * v.du * 16 * (uint64_t)N;
}

bool overlaps(const void* a, uint64_t na, const void* b, uint64_t nb) {
  if (na == 0 || nb == 0) return false;
  const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
  return x < y + nb && y < x + na;
}

// DV_ERR_HIP for a failed runtime call; with DV_DEBUG set in the environment
// the runtime's error name is also printed to stderr.
int hip_fail(hipError_t e, const char* what) {
  if (e == hipSuccess) return DV_OK;
  static const bool debug = getenv("DV_DEBUG") != nullptr;
  if (debug) fprintf(stderr, "libdv: %s failed: %s\n", what, hipGetErrorName(e));
  return DV_ERR_HIP;
}

int hip_status(hipError_t e) { return hip_fail(e, "hipMemcpy2DAsync"); }

// Whether [p, p + n) overlaps a paged view's block table, which the kernels
// read while the call writes: the table must stay out of everything written.
bool overlaps_table(const View& v, const void* p, uint64_t n) {
  return v.bt && overlaps(p, n, v.bt, (uint64_t)v.B * v.max_blocks * 4);
}

// Blocks of the table that hold tokens [t0, t0 + n).
int64_t blocks_of(const View& v, int64_t t0, int64_t n) {
  return n > 0 ? (t0 + n + v.bs - 1) / v.bs - t0 / v.bs : 0;
}

// Whether a paged stream-in with an owner-map workspace scatters in pool
// order: at most kPoolSeqMax sequences (their ranges travel in the launch's
// arguments), at least five ninths of the pool's blocks written, and every
// count inside the kernels' 32-bit arithmetic.  Pool order launches a
// workgroup for every block, and one that finds nothing to write still costs
// its launch and owner lookup: on MI355X, for the LLaMA-2-70B pool, pool
// order lost 4 % to table order with 47 % of the blocks written and 1 % with
// 52 %, broke even near 54 % and won 1.5 % at 57 %, 3 % at 62 % and 7 % at
// 95 %.
bool pool_order_applies(const View& v, const std::vector<int32_t>& t0,
                        const std::vector<int32_t>& n, int64_t N) {
  // 2^30 blocks: a tile's block numbers reach past the pool's last.
  if (v.B > dv::kPoolSeqMax || N >= (1ll << 31) || v.NB >= (1ll << 30) ||
      v.B * v.max_blocks >= (1ll << 31))
    return false;
  int64_t blocks = 0;
  for (int64_t b = 0; b < v.B; ++b) blocks += blocks_of(v, t0[b], n[b]);
  return 9 * blocks >= 5 * v.NB;
}

// Fills a launch's sequence table for sequences [g0, g0 + nseq) of the call;
// items(i) is the number of work items of sequence g0 + i.  Returns the sum of
// the items; the table holds it in 32 bits, which is enough for any grid that a
// launch accepts (below kMaxGroups workgroups).
template <int N, typename Items>
int64_t fill_seqs(dv::SeqTable<N>* s, const std::vector<int32_t>& t0,
                  const std::vector<int32_t>& n, int64_t g0, int nseq, Items items) {
  int64_t total = 0, tok = 0;
  for (int i = 0; i < N; ++i) {
    s->item[i] = i < nseq ? (int32_t)total : INT32_MAX;
    s->tok[i] = (int32_t)tok;
    s->t0[i] = i < nseq ? t0[g0 + i] : 0;
    if (i < nseq) {
      total += items(i);
      tok += n[g0 + i];
    }
  }
  s->tok[N] = (int32_t)tok;
  return total;
}

// The owner map of a whole call of at most N sequences in one launch.
template <int N>
hipError_t launch_owner_map(const View& v, const std::vector<int32_t>& t0,
                            const std::vector<int32_t>& n, hipStream_t st) {
  dv::OwnerMapArgs<N> a;
  memset(&a, 0, sizeof a);
  a.owner = v.owner;
  a.bt = v.bt;
  a.num_blocks = (int32_t)v.NB;
  a.max_blocks = (int32_t)v.max_blocks;
  a.d_bs = dv::fast_div((uint32_t)v.bs);
  a.chunks = (int32_t)fill_seqs(&a.s, t0, n, 0, (int)v.B, [&](int i) {
    return (blocks_of(v, t0[i], n[i]) + 63) / 64;
  });
  return dv::launch_owner_map<N>(a, st);
}

// The owner map of a whole call: one launch for a small table, else one
// clearing launch and one building launch per group of 64 sequences.
int build_owner_map(const View& v, const std::vector<int32_t>& t0, const std::vector<int32_t>& n,
                    hipStream_t st) {
  int64_t chunks = 0;
  for (int64_t b = 0; b < v.B; ++b) chunks += (blocks_of(v, t0[b], n[b]) + 63) / 64;
  const int64_t launches = 1 + (v.B + kSeqPerLaunch - 1) / kSeqPerLaunch;
  if (v.B <= dv::kSeqMany && chunks <= dv::kOwnerChunks * launches)
    return hip_fail(v.B <= kSeqPerLaunch ? launch_owner_map<kSeqPerLaunch>(v, t0, n, st)
                                         : launch_owner_map<dv::kSeqMany>(v, t0, n, st),
                    "owner map launch");
  dv::OwnerArgs o;
  memset(&o, 0, sizeof o);
  o.owner = v.owner;
  o.bt = v.bt;
  o.block_size = (int32_t)v.bs;
  o.num_blocks = (int32_t)v.NB;
  o.max_blocks = (int32_t)v.max_blocks;
  hipError_t e = dv::launch_owner_clear(o, st);
  if (e != hipSuccess) return hip_fail(e, "owner map launch");
  for (int64_t g0 = 0; g0 < v.B; g0 += kSeqPerLaunch) {
    o.nseq = (int32_t)std::min<int64_t>(kSeqPerLaunch, v.B - g0);
    o.b0 = (int32_t)g0;
    memset(&o.r, 0, sizeof o.r);
    bool any = false;
    for (int i = 0; i < o.nseq; ++i) {
      o.r.t0[i] = t0[g0 + i];
      o.r.n[i] = n[g0 + i];
      any = any || n[g0 + i] > 0;
    }
    if (!any) continue;
    e = dv::launch_owner_build(o, st);
    if (e != hipSuccess) return hip_fail(e, "owner map launch");
  }
  return DV_OK;
}

// The smallest power of two of tiles per workgroup for which the launch has
// fewer than kMaxGroups workgroups per slab, fill(steps) of them (at least one
// for each of its sequences, of which there are fewer than that).
template <typename Fill>
int32_t steps_for(Fill fill, int64_t* tiles) {
  int32_t steps = 1;
  while ((*tiles = fill(steps)) >= dv::kMaxGroups) steps *= 2;
  return steps;
}

// One launch over sequences [g0, g0 + nseq) of a call, their part of the
// contiguous buffer at `wire`.  In pool order (the owner map built) it covers
// the whole pool and all sequences of the call.
template <int N>
hipError_t launch_paged_group(int dir, bool pool, const View& v, int32_t l0, uint32_t nl,
                              const std::vector<int32_t>& t0, const std::vector<int32_t>& n,
                              int64_t g0, int nseq, int64_t w_slab, void* wire,
                              hipStream_t st) {
  const int64_t s_blk = v.H * v.bs * v.du, s_slab = v.NB * s_blk;
  int64_t tiles = 0;
  dv::PagedArgs<N> a;
  memset(&a, 0, sizeof a);
  a.pool = v.base;
  a.wire = wire;
  a.bt = v.bt + g0 * v.max_blocks;
  a.owner = pool ? v.owner : nullptr;
  a.s_slab = s_slab;
  a.s_blk = s_blk;
  a.m = {2 * l0, 0, w_slab};
  a.ub = (int32_t)(v.bs * v.du);
  a.du = (int32_t)v.du;
  a.heads = (int32_t)v.H;
  a.nseq = nseq;
  a.num_blocks = (int32_t)v.NB;
  a.max_blocks = (int32_t)v.max_blocks;
  a.d_ub = dv::fast_div((uint32_t)(v.bs * v.du));
  a.d_heads = dv::fast_div((uint32_t)v.H);
  a.d_bs = dv::fast_div((uint32_t)v.bs);
  a.d_max = dv::fast_div((uint32_t)v.max_blocks);
  int64_t units = 0;  // the longest array that tiles number through
  a.steps = steps_for(
      [&](int64_t steps) {
        const int64_t tile = dv::kPagedTile * steps;
        units = 0;
        const int64_t table = fill_seqs(&a.s, t0, n, g0, nseq, [&](int i) {
          const int64_t f = blocks_of(v, t0[g0 + i], n[g0 + i]) * s_blk;
          units = std::max(units, f);
          return (f + tile - 1) / tile;
        });
        if (!pool) return table;
        units = s_slab;
        return (s_slab + tile - 1) / tile;
      },
      &tiles);
  a.tiles = (int32_t)tiles;
  a.d_tiles = dv::fast_div((uint32_t)tiles);
  const bool wide = a.steps > 1 || units + dv::kPagedTile >= (1ll << 31) ||
                    tiles * 2 * nl >= (1ll << 31);
  return dv::launch_paged<N>(dir, a, wide, 2 * nl, st);
}

// A paged stream of runs longer than the short-run kernel's, in launches of
// at most N sequences.
template <int N>
int run_paged(int dir, bool pool, const View& v, int32_t l0, uint32_t nl,
              const std::vector<int32_t>& t0, const std::vector<int32_t>& n, int64_t w_slab,
              void* wire, hipStream_t st) {
  int64_t p = 0;  // tokens of all earlier launches
  for (int64_t g0 = 0; g0 < v.B; g0 += N) {
    const int nseq = (int)std::min<int64_t>(N, v.B - g0);
    int64_t tok = 0;
    for (int i = 0; i < nseq; ++i) tok += n[g0 + i];
    if (tok == 0) continue;
    const hipError_t e =
        launch_paged_group<N>(dir, pool, v, l0, nl, t0, n, g0, nseq, w_slab,
                              static_cast<char*>(wire) + (uint64_t)p * v.H * v.du * 16, st);
    if (e != hipSuccess) return hip_fail(e, "paged kernel launch");
    p += tok;
  }
  return DV_OK;
}

// Lists, from sequence *b on, up to N sequences that have tokens and whose rows
// of `row` units each count below 2^31 units, and moves *b past them.  Returns
// their number; *tok is their tokens, *even whether they have equally many.
template <int N, typename Args>
int fill_rows(Args* a, const std::vector<int32_t>& t0, const std::vector<int32_t>& n, int64_t row,
              int64_t* b, int64_t* tok, bool* even) {
  int nseq = 0;
  *tok = 0;
  *even = true;
  for (; *b < (int64_t)n.size() && nseq < N; ++*b) {
    const int32_t k = n[*b];
    if (k == 0) continue;
    if ((*tok + k) * row >= (1ll << 31)) break;
    a->tok[nseq] = (int32_t)*tok;
    a->t0[nseq] = t0[*b];
    a->seq[nseq] = (int32_t)*b;
    *tok += k;
    *even = *even && k * (int64_t)(nseq + 1) == *tok;
    ++nseq;
  }
  a->tok[nseq] = (int32_t)*tok;
  for (int i = nseq + 1; i <= N; ++i) a->tok[i] = INT32_MAX;
  a->total = (int32_t)(*tok * row);
  return nseq;
}

// A stream of short runs (or any whose slabs hold fewer than 2^31 units), in
// launches of at most N sequences that have tokens and fewer than 2^31 units.
template <int N>
int run_rows(int dir, const View& v, int32_t l0, uint32_t nl, const std::vector<int32_t>& t0,
             const std::vector<int32_t>& n, int64_t w_slab, void* wire, hipStream_t st) {
  dv::RowArgs<N> a;
  memset(&a, 0, sizeof a);
  a.cache = v.base;
  a.bt = v.bt;
  a.m = {2 * l0, 0, w_slab};
  a.du = (int32_t)v.du;
  a.heads = (int32_t)v.H;
  a.d_du = dv::fast_div((uint32_t)v.du);
  a.d_heads = dv::fast_div((uint32_t)v.H);
  a.d_bs = dv::fast_div(1);
  for (int half = 0; half < 2; ++half) {
    a.s_tok[half] = v.du;
    a.s_e[half] = 1;
  }
  if (v.kind == DV_PAGED) {
    a.paged = 1;
    a.block_size = (int32_t)v.bs;
    a.num_blocks = (int32_t)v.NB;
    a.max_blocks = (int32_t)v.max_blocks;
    a.s_slab = v.NB * v.H * v.bs * v.du;
    a.s_b = v.H * v.bs * v.du;
    a.s_h = v.bs * v.du;
    a.d_bs = dv::fast_div((uint32_t)v.bs);
  } else {
    a.s_slab = v.B * v.H * v.S * v.du;
    a.s_b = v.H * v.S * v.du;
    a.s_h = v.S * v.du;
    if (v.kind == DV_DENSE_KSPLIT) {  // key slabs: groups S units apart, tokens 1
      a.s_tok[0] = 1;
      a.s_e[0] = v.S;
    }
  }
  const int32_t max_n = *std::max_element(n.begin(), n.end());
  a.tile = (int32_t)std::max<int64_t>(1, dv::kThreads * dv::kRowsUnroll / v.du);
  a.d_tile = dv::fast_div((uint32_t)a.tile);
  const int64_t row = v.H * v.du;  // units of one token
  int64_t p = 0;                   // tokens of all earlier launches
  for (int64_t b = 0; b < v.B;) {
    int64_t tok;
    bool even;
    const int nseq = fill_rows<N>(&a, t0, n, row, &b, &tok, &even);
    if (nseq == 0) continue;  // only sequences without tokens were left
    a.wire = static_cast<char*>(wire) + (uint64_t)p * row * 16;
    a.n = (int32_t)(tok / nseq);  // read where the runs are even
    a.d_seq = dv::fast_div((uint32_t)(v.H * a.n));
    a.d_n = dv::fast_div((uint32_t)a.n);
    // Key slabs through LDS from 4 MB on; smaller launches are bound by
    // latency (1.9 MB: 3.1 us out against 2.7 without, 4.2 in against 4.3).
    const bool split = v.kind == DV_DENSE_KSPLIT && max_n > 1 &&
                       (int64_t)a.total * 2 * nl >= (1 << 18);
    const hipError_t e = split ? dv::launch_split_rows<N>(dir, a, 2 * nl, st)
                               : dv::launch_rows<N>(dir, even, a, 2 * nl, st);
    if (e != hipSuccess) return hip_fail(e, "short-run kernel launch");
    p += tok;
  }
  return DV_OK;
}

// A dense stream of runs longer than the short-run kernel's, in launches of at
// most N sequences.
template <int N>
int run_dense(int dir, const View& v, int32_t l0, uint32_t nl, const std::vector<int32_t>& t0,
              const std::vector<int32_t>& n, bool eighths, int64_t w_slab, void* wire,
              hipStream_t st) {
  dv::DenseRunArgs<N> a;
  memset(&a, 0, sizeof a);
  a.s_slab = v.B * v.H * v.S * v.du;
  a.s_b = v.H * v.S * v.du;
  a.s_h = v.S * v.du;
  a.m = {2 * l0, 0, w_slab};
  a.du = (int32_t)v.du;
  a.heads = (int32_t)v.H;
  int64_t p = 0;  // tokens of all earlier launches
  for (int64_t g0 = 0; g0 < v.B; g0 += N) {
    const int nseq = (int)std::min<int64_t>(N, v.B - g0);
    const int64_t tiles = fill_seqs(&a.s, t0, n, g0, nseq, [&](int i) {
      return v.H * ((n[g0 + i] * v.du + dv::kDenseTile - 1) / dv::kDenseTile);
    });
    if (tiles == 0) continue;
    a.cache = v.base + (uint64_t)(g0 * a.s_b) * 16;
    a.wire = static_cast<char*>(wire) + (uint64_t)p * v.H * v.du * 16;
    a.deal = dv::deal_of(tiles, 2 * nl, eighths);
    const hipError_t e = dv::launch_dense_runs<N>(dir, a, 2 * nl, st);
    if (e != hipSuccess) return hip_fail(e, "dense kernel launch");
    p += a.s.tok[N];
  }
  return DV_OK;
}

// A split-key stream of runs longer than the short-run kernel's, in launches
// of at most N sequences.
template <int N>
int run_split(int dir, const View& v, int32_t l0, uint32_t nl, const std::vector<int32_t>& t0,
              const std::vector<int32_t>& n, int64_t w_slab, void* wire, hipStream_t st) {
  dv::SplitArgs<N> a;
  memset(&a, 0, sizeof a);
  a.cache = v.base;
  a.s_slab = v.B * v.H * v.S * v.du;
  a.s_b = v.H * v.S * v.du;
  a.s_h = v.S * v.du;
  a.m = {2 * l0, 0, w_slab};
  a.du = (int32_t)v.du;
  a.heads = (int32_t)v.H;
  a.seq_cap = (int32_t)v.S;
  int units = dv::split_units(v.du);
  if (v.S % 8 == 0) {  // then slabs, heads and groups are whole lines apart
    a.line0 = (int32_t)((reinterpret_cast<uintptr_t>(v.base) >> 4) & 7);
    a.line_mask = 7;
  } else if (dir == dv::kUnpack && units == 2 && v.du >= dv::kSplitEightDu &&
             w_slab * 2 * nl >= dv::kSplitEightMin) {
    // Eight units per lane save a ninth of the time that two take, but a run of
    // several tiles loses three quarters of a small tile's time to its last one.
    const int64_t small = dv::split_tile(v.du, 2), tile = dv::split_tile(v.du, 8);
    int64_t tok = 0, smalls = 0, tiles = 0, several = 0;
    for (int32_t k : n) {
      tok += k;
      smalls += (k + small - 1) / small;
      tiles += (k + tile - 1) / tile;
      several += k > tile;
    }
    if (3 * tok >= tiles * tile && 11 * smalls > 75 * several) units = 8;
  }
  a.tile = dv::split_tile(v.du, units);
  a.d_du = dv::fast_div((uint32_t)v.du);
  a.d_tile = dv::fast_div((uint32_t)a.tile);
  int64_t p = 0;  // tokens of all earlier launches
  for (int64_t g0 = 0; g0 < v.B; g0 += N) {
    const int nseq = (int)std::min<int64_t>(N, v.B - g0);
    const int64_t tiles = fill_seqs(&a.s, t0, n, g0, nseq, [&](int i) {
      const int64_t lead = (a.line0 + t0[g0 + i]) & a.line_mask, k = n[g0 + i];
      return k > 0 ? v.H * ((lead + k + a.tile - 1) / a.tile) : 0;
    });
    if (tiles == 0) continue;
    a.wire = static_cast<char*>(wire) + (uint64_t)p * v.H * v.du * 16;
    a.b0 = (int32_t)g0;
    a.deal = dv::deal_of(tiles, 2 * nl, true);
    const hipError_t e = dv::launch_split<N>(dir, a, 2 * nl, st);
    if (e != hipSuccess) return hip_fail(e, "split-key kernel launch");
    p += a.s.tok[N];
  }
  return DV_OK;
}

// The largest calls the boundary takes, as the header counts them: over any 64
// consecutive sequences (from the first, the 65th, ...) fewer than 2^31 16-byte
// units of one slab for runs of at most kSmallRunUnits, else fewer than 2^31
// pieces: 512 units of a dense or split-key run, 64 tokens of a split-key one,
// two heads of a paged block.  The pieces are those of no present kernel: the
// limit is the caller's, whatever tiles a launch uses, and stays where it is.
// Launches hold up to 256 sequences and count for themselves: rows and copies
// below 2^31 units each (fill_rows; one token of 256 sequences is below 2^28),
// paged tiles below kMaxGroups (steps_for), dense and split-key tiles likewise,
// or else 64 sequences to a launch, which dv_kernels.hip refuses where even those
// are too many for a grid.
bool within_limits(const View& v, const std::vector<int32_t>& t0, const std::vector<int32_t>& n,
                   bool small) {
  constexpr int64_t kPieceUnits = 512, kPieceTokens = 64, kPieceHeads = 2;
  for (int64_t g0 = 0; g0 < v.B; g0 += kSeqPerLaunch) {
    int64_t pieces = 0, by_token = 0;
    for (int64_t b = g0; b < std::min<int64_t>(g0 + kSeqPerLaunch, v.B); ++b) {
      const int64_t k = n[b];
      if (small)
        pieces += k * v.H * v.du;
      else if (v.kind == DV_PAGED)
        pieces += blocks_of(v, t0[b], k) * ((v.H + kPieceHeads - 1) / kPieceHeads);
      else
        pieces += v.H * ((k * v.du + kPieceUnits - 1) / kPieceUnits);
      if (!small && v.kind == DV_DENSE_KSPLIT)
        by_token += v.H * ((k + kPieceTokens - 1) / kPieceTokens);
    }
    if (std::max(pieces, by_token) >= (1ll << 31)) return false;
  }
  return true;
}

// Enqueue the pack (dir = kPack) or unpack of the validated ranges.  The wire
// is at `wire`; per (layer, K|V) slab it holds N*H*du units.
int run_stream(int dir, const View& v, int32_t l0, int32_t l1, const std::vector<int32_t>& t0,
               const std::vector<int32_t>& n, int64_t N, void* wire, hipStream_t st) {
  if (N == 0 || l1 == l0) return DV_OK;
  const int64_t w_slab = N * v.H * v.du;
  const uint32_t nl = (uint32_t)(l1 - l0);
  int32_t max_n = 0;
  for (int32_t x : n) max_n = std::max(max_n, x);
  const bool single = max_n <= 1;
  // Runs of at most kSmallRunUnits units per (sequence, head) go through the
  // flattened short-run kernel instead of the tiled ones.
  const bool small = !single && (int64_t)max_n * v.du <= kSmallRunUnits;

  if (!single && !within_limits(v, t0, n, small)) return DV_ERR_UNSUPPORTED;

  bool flat = single || small;  // the short-run kernel
  if (v.kind == DV_PAGED && !single && !small) {
    // Tiles over whole blocks leave the lanes of tokens outside the range
    // idle: where the range fills less than three quarters of its blocks, rows.
    // Tiles in table order, tiles in pool order, rows; 20 layers, 8 heads x 128
    // x 2 bytes, 32 sequences, the pool written whole: blocks of 16 tokens 36 %
    // full 17.9, -, 13.8 us out, 17.9, 18.8, 14.3 in; 73 % 55.2, -, 53.1 out,
    // 55.5, 55.7, 54.2 in; 94 % 54.7, -, 54.1 out, 55.3, 55.4, 54.6 in; of 64
    // tokens 71 % full 191, -, 182 out, 192, 187, 191 in, 90 % 278, -, 278 out,
    // 282, 276, 292 in; of 256 tokens 34 % 205, -, 142 out, 209, 168, 151 in.
    int64_t blocks = 0;
    for (int64_t b = 0; b < v.B; ++b) blocks += blocks_of(v, t0[b], n[b]);
    const bool partial = 4 * N < 3 * blocks * v.bs;
    flat = partial && w_slab < (1ll << 31);
    const bool pool =
        !partial && dir == dv::kUnpack && v.owner && pool_order_applies(v, t0, n, N);
    if (pool) {
      const int rc = build_owner_map(v, t0, n, st);
      if (rc != DV_OK) return rc;
    }
    // More than 64 sequences go 256 to a launch while their tokens count
    // below 2^31 (those of 64 always do).
    if (!flat)
      return v.B > kSeqPerLaunch && N < (1ll << 31)
                 ? run_paged<dv::kSeqMany>(dir, pool, v, l0, nl, t0, n, w_slab, wire, st)
                 : run_paged<kSeqPerLaunch>(dir, pool, v, l0, nl, t0, n, w_slab, wire, st);
  }

  if (v.kind == DV_DENSE_KSPLIT && !flat) {
    // Where tiles of one head each would be less than three quarters full, rows
    // across heads and sequences: always on the way out (up to 22 tokens of 16
    // groups 44 us by tiles, 32 by rows), on the way in up to 1.6 GB over the
    // groups per token.  A workgroup's rows of a key slab are written in pieces of
    // lines, the shorter the wider the tokens, and past the caches those cost what
    // whole lines do.  Tiles and rows, 64 sequences: 32 groups, 10-20 tokens, 10 MB
    // 7.4 and 6.6 us, 20 MB 12.2 and 12.8, 60 MB 30.7 and 35.6, 391 MB 184 and 230;
    // 16 groups, 10-60 tokens, 24 MB 11.7 and 12.4, 96 MB 40.8 and 45.8, 379 MB 147
    // and 181, 33 tokens, 110 MB 52.8 and 44.6; 10 groups, 62 tokens, 77 MB 37.3 and
    // 32.5; 8 groups, 23-47 tokens, 106 MB 43.8 and 45.2, 393 MB 156 and 177; 3
    // groups, 102 tokens, 366 MB 135 and 123.  Emptier tiles lose again, 400 MB: 8
    // groups, 37 % full 203 and 191, 44 % 174 and 185; 12 groups, 33 % 240 and 232,
    // 41 % 206 and 215; 16 groups, 29 % 256 and 248, 41 % 198 and 229; 24 groups,
    // 17 % 287 and 252, 25 % 212 and 230; 32 groups, 32 % 246 and 277.
    const int64_t tile = dv::split_tile(v.du, dv::split_units(v.du));
    int64_t tiles = 0;
    for (int64_t b = 0; b < v.B; ++b) tiles += (n[b] + tile - 1) / tile;
    flat = 4 * N < 3 * tiles * tile && w_slab < (1ll << 31) &&
           (dir == dv::kPack || v.du < 8 || w_slab * 2 * nl * v.du <= 100'000'000 ||
            80 * N < (40 - v.du) * tiles * tile);
    if (!flat)
      return v.B > kSeqPerLaunch && N < (1ll << 31) &&
                     (tiles + v.B) * v.H < dv::kMaxGroups
                 ? run_split<dv::kSeqMany>(dir, v, l0, nl, t0, n, w_slab, wire, st)
                 : run_split<kSeqPerLaunch>(dir, v, l0, nl, t0, n, w_slab, wire, st);
  }
  bool eighths = true;
  int64_t dense_tiles = 0;
  if (v.kind == DV_DENSE && !flat) {
    // Runs of a few hundred units fill their last tile badly.  A pack goes by
    // rows then (its writes stay contiguous), an unpack only where most of
    // the lanes would idle, and its tiles are not dealt in eighths.  Tiles in
    // eighths, tiles in the hardware's order, rows: 11 sequences of 1-47
    // tokens, 45 heads x 128 x 2 bytes, 33 layers (55 % full) 77.5, 71, 68.5 us
    // out, 77.8, 73.5, 77.4 in; 13 of 1-18 tokens, 3 heads (30 %) 6.5, -, 5.3
    // out, 7.6, -, 4.9 in; 60 of 24-472 tokens, 8 heads x 80 (91 %) 729, 799,
    // 716 out, 728, 814, 792 in; prompts of 64-2048 tokens (98 %) 389, 416, 398
    // out, 390, 423, 434 in.  Tokens of one unit are a look-up each: below 16 MB
    // their packs keep tiles that are 70 % full (8 MB, 79 %: 4.5 us by tiles, 5.3
    // by rows; 11 MB, 74 % 5.6 and 6.1, 66 % 6.0 and 6.1, 52 % 7.5 and 6.4; 33 MB,
    // 78 % 13.3 and 13.6, 82 % 14.6 and 14.1; four units a token, 11 MB, 78 % 5.7
    // and 5.2).
    for (int64_t b = 0; b < v.B; ++b)
      dense_tiles += v.H * ((n[b] * v.du + dv::kDenseTile - 1) / dv::kDenseTile);
    const int64_t full = dense_tiles * dv::kDenseTile;
    const bool look_ups = v.du == 1 && w_slab * 2 * nl < (1 << 20);
    const int line = dir == dv::kUnpack ? 45 : look_ups ? 70 : 92;
    flat = w_slab < (1ll << 31) && 100 * w_slab < line * full;
    eighths = 100 * w_slab >= 80 * full;
  }
  if (flat)
    return v.B > kSeqPerLaunch ? run_rows<dv::kSeqMany>(dir, v, l0, nl, t0, n, w_slab, wire, st)
                               : run_rows<kSeqPerLaunch>(dir, v, l0, nl, t0, n, w_slab, wire, st);
  return v.B > kSeqPerLaunch && N < (1ll << 31) && dense_tiles < dv::kMaxGroups
             ? run_dense<dv::kSeqMany>(dir, v, l0, nl, t0, n, eighths, w_slab, wire, st)
             : run_dense<kSeqPerLaunch>(dir, v, l0, nl, t0, n, eighths, w_slab, wire, st);
}

int check_kind_supported(const View& v) {
  if (v.kind == DV_DENSE_KSPLIT && (16 % v.E != 0 || v.du > dv::kKsplitMaxDu))
    return DV_ERR_UNSUPPORTED;
  return DV_OK;
}

int stream_out(const dv_cache* src, int32_t mb, int32_t l0, int32_t l1, const int32_t* t0,
               const int32_t* t1, void* dst, uint64_t dst_cap, uint64_t* out_bytes,
               void* stream) {
  View v;
  int rc = view_of(src, mb, &v);
  if (rc != DV_OK) return rc;
  std::vector<int32_t> r0, rn;
  int64_t N = 0;
  rc = ranges_of(v, l0, l1, t0, t1, &r0, &rn, &N);
  if (rc != DV_OK) return rc;
  const uint64_t need = wire_bytes(v, l0, l1, N);
  if (out_bytes) *out_bytes = need;
  if (need > dst_cap) return DV_ERR_SPACE;
  if (need == 0) return DV_OK;
  if (!dst || !aligned16(dst)) return DV_ERR_INVALID;
  if (overlaps(dst, need, v.base, v.bytes) || overlaps_table(v, dst, need))
    return DV_ERR_INVALID;
  rc = check_kind_supported(v);
  if (rc != DV_OK) return rc;
  return run_stream(dv::kPack, v, l0, l1, r0, rn, N, dst, static_cast<hipStream_t>(stream));
}

// The validated ranges of narrow rows between two dense caches by kernel, in
// launches of at most N sequences that have tokens and fewer than 2^31 units.
template <int N>
int run_copy(const View& from, const View& to, int32_t l0, uint32_t nl,
             const std::vector<int32_t>& t0, const std::vector<int32_t>& n, hipStream_t st) {
  dv::CopyArgs<N> a;
  memset(&a, 0, sizeof a);
  a.src = from.base;
  a.dst = to.base;
  a.s_slab = from.B * from.H * from.S * from.du;
  a.s_b = from.H * from.S * from.du;
  a.s_h = from.S * from.du;
  a.d_slab = to.B * to.H * to.S * to.du;
  a.d_b = to.H * to.S * to.du;
  a.d_h = to.S * to.du;
  a.slab0 = 2 * l0;
  a.du = (int32_t)from.du;
  a.heads = (int32_t)from.H;
  a.d_du = dv::fast_div((uint32_t)from.du);
  a.d_heads = dv::fast_div((uint32_t)from.H);
  for (int64_t b = 0; b < from.B;) {
    int64_t tok;
    bool even;
    if (fill_rows<N>(&a, t0, n, from.H * from.du, &b, &tok, &even) == 0) continue;
    const hipError_t e = dv::launch_copy<N>(a, 2 * nl, st);
    if (e != hipSuccess) return hip_fail(e, "copy kernel launch");
  }
  return DV_OK;
}

// Copy rows of the validated ranges between two dense caches with DMA.
int swap_copy(const dv_cache* from, int32_t from_mb, const dv_cache* to, int32_t to_mb,
              int32_t l0, int32_t l1, const int32_t* t0, const int32_t* t1, void* stream,
              int from_mem, int to_mem) {
  View a, b;
  int rc = view_of(from, from_mb, &a);
  if (rc != DV_OK) return rc;
  rc = view_of(to, to_mb, &b);
  if (rc != DV_OK) return rc;
  if (a.kind != DV_DENSE || b.kind != DV_DENSE) return DV_ERR_UNSUPPORTED;
  if (a.L != b.L || a.H != b.H || a.D != b.D || a.B != b.B || a.E != b.E) return DV_ERR_INVALID;
  if (a.mem != from_mem || b.mem != to_mem) return DV_ERR_INVALID;
  std::vector<int32_t> r0, rn;
  int64_t N = 0;
  rc = ranges_of(a, l0, l1, t0, t1, &r0, &rn, &N);
  if (rc != DV_OK) return rc;
  for (int64_t i = 0; i < b.B; ++i)
    if ((int64_t)r0[i] + rn[i] > b.cap) return DV_ERR_RANGE;
  if (overlaps(a.base, a.bytes, b.base, b.bytes)) return DV_ERR_INVALID;
  if (N == 0 || l1 == l0) return DV_OK;

  hipStream_t st = static_cast<hipStream_t>(stream);
  int32_t max_n = 0;
  for (int32_t x : rn) max_n = std::max(max_n, x);
  if ((int64_t)max_n * a.du * 16 < kNarrowRowBytes) {
    // Narrow rows (a decode step's update): one kernel copies them straight
    // between the slot and the pinned mirror; DMA would take one descriptor
    // per row (or one call per row block when the ranges are ragged).
    // Every launch group's grid is checked before anything is enqueued.
    for (int64_t g0 = 0; g0 < a.B; g0 += kSeqPerLaunch) {
      int64_t units = 0;
      for (int64_t b = g0; b < std::min<int64_t>(g0 + kSeqPerLaunch, a.B); ++b)
        units += (int64_t)rn[b] * a.H * a.du;
      if (units >= (1ll << 31)) return DV_ERR_UNSUPPORTED;
    }
    const uint32_t nl = (uint32_t)(l1 - l0);
    return a.B > kSeqPerLaunch ? run_copy<dv::kSeqMany>(a, b, l0, nl, r0, rn, st)
                               : run_copy<kSeqPerLaunch>(a, b, l0, nl, r0, rn, st);
  }

  const hipMemcpyKind kind =
      from_mem == DV_MEM_DEVICE ? hipMemcpyDeviceToHost : hipMemcpyHostToDevice;
  const size_t tok = (size_t)a.du * 16;
  const size_t ap = (size_t)a.S * tok, bp = (size_t)b.S * tok;  // row pitches
  bool uniform = true;
  for (int64_t i = 1; i < a.B; ++i)
    if (r0[i] != r0[0] || rn[i] != rn[0]) uniform = false;
  if (uniform) {
    // Rows (slab, b, h) of the layer range are consecutive at one pitch.
    const size_t row0 = (size_t)2 * l0 * a.B * a.H;
    const size_t rows = (size_t)2 * (l1 - l0) * a.B * a.H;
    return hip_status(hipMemcpy2DAsync(b.base + row0 * bp + r0[0] * tok, bp,
                                       a.base + row0 * ap + r0[0] * tok, ap, rn[0] * tok, rows,
                                       kind, st));
  }
  // Ragged ranges: one 3-D copy per sequence, its heads' rows of every slab.
  // A 2-D copy per (slab, sequence) costs its 10 to 25 us that much more often:
  // 16 sequences of 24-86 KB rows, 12 slabs (42 MB) took 2.5 ms one way against
  // 0.90, 2 sequences of 340 KB rows, 16 slabs (177 MB) 3.41 against 3.12.
  // Slabs of 2 GB and more keep the 2-D copies: a slab is the copy's slice.
  const size_t slab_rows = (size_t)a.B * a.H;
  const bool slices = slab_rows * std::max(ap, bp) < (1ull << 31);
  for (int64_t s = 0; s < a.B; ++s) {
    if (rn[s] == 0) continue;
    const size_t width = (size_t)rn[s] * tok, at = (size_t)r0[s] * tok;
    for (int64_t slab = 2 * l0; slab < 2 * l1; ++slab) {
      const size_t row0 = (size_t)(slab * a.B + s) * a.H;
      char* from_row = a.base + row0 * ap + at;
      char* to_row = b.base + row0 * bp + at;
      if (slices) {
        hipMemcpy3DParms p;
        memset(&p, 0, sizeof p);
        p.srcPtr = make_hipPitchedPtr(from_row, ap, width, slab_rows);
        p.dstPtr = make_hipPitchedPtr(to_row, bp, width, slab_rows);
        p.extent = make_hipExtent(width, (size_t)a.H, (size_t)(2 * (l1 - l0)));
        p.kind = kind;
        const hipError_t e = hipMemcpy3DAsync(&p, st);
        if (e != hipSuccess) return hip_fail(e, "hipMemcpy3DAsync");
        break;  // every slab of this sequence
      }
      const hipError_t e =
          hipMemcpy2DAsync(to_row, bp, from_row, ap, width, (size_t)a.H, kind, st);
      if (e != hipSuccess) return hip_fail(e, "hipMemcpy2DAsync");
    }
  }
  return DV_OK;
}

}  // namespace

namespace dv {

hipError_t create_side_streams(hipStream_t* shared_queue, hipStream_t* own_queue) {
  *shared_queue = *own_queue = nullptr;
  hipError_t e = hipStreamCreateWithFlags(shared_queue, hipStreamNonBlocking);
  if (e != hipSuccess) return e;
  int device = 0, cus = 0;
  e = hipGetDevice(&device);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device);
  if (e != hipSuccess || cus <= 0) return e != hipSuccess ? e : hipErrorInvalidDevice;
  std::vector<uint32_t> mask((cus + 31) / 32, 0xffffffffu);  // every CU
  if (cus % 32) mask.back() = (1u << (cus % 32)) - 1u;
  return hipExtStreamCreateWithCUMask(own_queue, (uint32_t)mask.size(), mask.data());
}

}  // namespace dv

extern "C" {

int dv_api_version(void) { return DV_API_VERSION; }

const char* dv_status_string(int status) {
  switch (status) {
    case DV_OK: return "ok";
    case DV_ERR_INVALID: return "invalid argument";
    case DV_ERR_RANGE: return "range outside the cache";
    case DV_ERR_SPACE: return "buffer too small";
    case DV_ERR_UNSUPPORTED: return "unsupported layout or size";
    case DV_ERR_HIP: return "HIP runtime error";
    default: return "unknown status";
  }
}

int dv_cache_bytes(const dv_cache* c, uint64_t* out_bytes) {
  View v;
  int rc = layout_of(c, &v);
  if (rc != DV_OK) return rc;
  if (out_bytes) *out_bytes = v.bytes;
  return DV_OK;
}

int dv_packed_bytes(const dv_cache* c, int32_t l0, int32_t l1, const int32_t* t0,
                    const int32_t* t1, uint64_t* out_bytes) {
  View v;
  int rc = layout_of(c, &v);
  if (rc != DV_OK) return rc;
  std::vector<int32_t> r0, rn;
  int64_t N = 0;
  rc = ranges_of(v, l0, l1, t0, t1, &r0, &rn, &N);
  if (rc != DV_OK) return rc;
  if (out_bytes) *out_bytes = wire_bytes(v, l0, l1, N);
  return DV_OK;
}

int dv_stream_out_prompt(const dv_cache* src, int32_t mb, int32_t l0, int32_t l1,
                         const int32_t* t0, const int32_t* t1, void* dst, uint64_t dst_cap,
                         uint64_t* out_bytes, void* stream) {
  return stream_out(src, mb, l0, l1, t0, t1, dst, dst_cap, out_bytes, stream);
}

int dv_stream_out_token(const dv_cache* src, int32_t mb, int32_t l0, int32_t l1,
                        const int32_t* pos, void* dst, uint64_t dst_cap, uint64_t* out_bytes,
                        void* stream) {
  if (!src || !pos || src->batch <= 0) return DV_ERR_INVALID;
  std::vector<int32_t> a(src->batch), e(src->batch);
  for (int32_t b = 0; b < src->batch; ++b) {
    if (pos[b] == INT32_MAX) return DV_ERR_RANGE;  // before pos + 1 is formed
    a[b] = pos[b] < 0 ? 0 : pos[b];
    e[b] = pos[b] < 0 ? 0 : pos[b] + 1;
  }
  return stream_out(src, mb, l0, l1, a.data(), e.data(), dst, dst_cap, out_bytes, stream);
}

}  // extern "C"

namespace dv {
int noalloc_owner_map(hipStream_t stream, int32_t** out);  // dv_noalloc.hip
}  // namespace dv

namespace {

// dv_stream_in, and with `noalloc` dv_stream_in_noalloc: a paged receiver's
// owner map then lives in the library's static per-device array instead of
// the caller's workspace.
int stream_in(const dv_cache* dst, int32_t mb, int32_t l0, int32_t l1, const int32_t* t0,
              const int32_t* t1, const void* src, uint64_t src_bytes, void* stream,
              bool noalloc) {
  dv_cache own;
  if (noalloc && dst) {
    own = *dst;
    own.block_owner = nullptr;  // the caller's workspace, if any, is ignored
    dst = &own;
  }
  View v;
  int rc = view_of(dst, mb, &v);
  if (rc != DV_OK) return rc;
  if (noalloc && v.kind == DV_PAGED && v.NB > DV_NOALLOC_MAX_BLOCKS) return DV_ERR_UNSUPPORTED;
  std::vector<int32_t> r0, rn;
  int64_t N = 0;
  rc = ranges_of(v, l0, l1, t0, t1, &r0, &rn, &N);
  if (rc != DV_OK) return rc;
  const uint64_t need = wire_bytes(v, l0, l1, N);
  if (src_bytes < need) return DV_ERR_SPACE;
  if (need == 0) return DV_OK;
  if (!src || !aligned16(src)) return DV_ERR_INVALID;
  if (overlaps(src, need, v.base, v.bytes) || overlaps_table(v, v.base, v.bytes))
    return DV_ERR_INVALID;
  if (v.owner && (overlaps(v.owner, (uint64_t)v.NB * 4, v.base, v.bytes) ||
                  overlaps(v.owner, (uint64_t)v.NB * 4, src, need) ||
                  overlaps_table(v, v.owner, (uint64_t)v.NB * 4)))
    return DV_ERR_INVALID;
  rc = check_kind_supported(v);
  if (rc != DV_OK) return rc;
  if (noalloc && v.kind == DV_PAGED) {
    rc = dv::noalloc_owner_map(static_cast<hipStream_t>(stream), &v.owner);
    if (rc != DV_OK) return rc;
  }
  return run_stream(dv::kUnpack, v, l0, l1, r0, rn, N, const_cast<void*>(src),
                    static_cast<hipStream_t>(stream));
}

}  // namespace

extern "C" {

int dv_stream_in(const dv_cache* dst, int32_t mb, int32_t l0, int32_t l1, const int32_t* t0,
                 const int32_t* t1, const void* src, uint64_t src_bytes, void* stream) {
  return stream_in(dst, mb, l0, l1, t0, t1, src, src_bytes, stream, false);
}

int dv_stream_in_noalloc(const dv_cache* dst, int32_t mb, int32_t l0, int32_t l1,
                         const int32_t* t0, const int32_t* t1, const void* src,
                         uint64_t src_bytes, void* stream) {
  return stream_in(dst, mb, l0, l1, t0, t1, src, src_bytes, stream, true);
}

int dv_block_claims(const dv_cache* c, int32_t mb, const int32_t* t0, const int32_t* t1,
                    int32_t* counts, void* stream) {
  View v;
  int rc = view_of(c, mb, &v);
  if (rc != DV_OK) return rc;
  if (v.kind != DV_PAGED) return DV_ERR_UNSUPPORTED;
  std::vector<int32_t> r0, rn;
  int64_t N = 0;
  rc = ranges_of(v, 0, (int32_t)v.L, t0, t1, &r0, &rn, &N);
  if (rc != DV_OK) return rc;
  if (!counts || (reinterpret_cast<uintptr_t>(counts) & 3u) != 0) return DV_ERR_INVALID;
  if (overlaps(counts, (uint64_t)v.NB * 4, v.base, v.bytes) ||
      overlaps_table(v, counts, (uint64_t)v.NB * 4))
    return DV_ERR_INVALID;
  hipStream_t st = static_cast<hipStream_t>(stream);
  for (int64_t g0 = 0; g0 < v.B; g0 += kSeqPerLaunch) {
    const int nseq = (int)std::min<int64_t>(kSeqPerLaunch, v.B - g0);
    dv::OwnerArgs o;
    memset(&o, 0, sizeof o);
    o.owner = counts;
    o.bt = v.bt;
    o.nseq = nseq;
    o.block_size = (int32_t)v.bs;
    o.num_blocks = (int32_t)v.NB;
    o.max_blocks = (int32_t)v.max_blocks;
    o.b0 = (int32_t)g0;
    for (int i = 0; i < nseq; ++i) {
      o.r.t0[i] = r0[g0 + i];
      o.r.n[i] = rn[g0 + i];
    }
    const hipError_t e = dv::launch_block_claims(o, g0 == 0, st);
    if (e != hipSuccess) return hip_fail(e, "block claims launch");
  }
  return DV_OK;
}

int dv_swap_out(const dv_cache* dev, int32_t slot, const dv_cache* host, int32_t host_mb,
                int32_t l0, int32_t l1, const int32_t* t0, const int32_t* t1, void* stream) {
  return swap_copy(dev, slot, host, host_mb, l0, l1, t0, t1, stream, DV_MEM_DEVICE,
                   DV_MEM_HOST_PINNED);
}

int dv_swap_in(const dv_cache* host, int32_t host_mb, const dv_cache* dev, int32_t slot,
               int32_t l0, int32_t l1, const int32_t* t0, const int32_t* t1, void* stream) {
  return swap_copy(host, host_mb, dev, slot, l0, l1, t0, t1, stream, DV_MEM_HOST_PINNED,
                   DV_MEM_DEVICE);
}

}  // extern "C"
