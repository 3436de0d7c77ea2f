// Planned persistent launches: append rows alone, or one rollout step's
// decode rows (one new token each) and append rows (a chunk of new
// observation tokens each) together, against their paged caches.
//
// A plan kernel (one workgroup) lists the append tiles (row, query block) of
// the call from the device-resident lengths: the rows sorted by the key blocks
// of their longest (last) tile, longest first (a counting sort), each row's
// query blocks last first. The attention kernel runs one workgroup of 8 waves
// per CU over them, in one of two ways.
//
// Queue mode (enough tiles to fill the chip): one queue per XCD; queue q takes
// KV heads q, q + 8, q + 16, ... of every tile. The long tiles start early and
// the short ones fill the end, and the tiles of one row and head follow each
// other, so that the CUs of an XCD walk the same pages of K/V at about the
// same time and share them through the XCD's L2. Workgroups are placed on the
// XCDs round robin, so workgroup w starts on queue w mod 8 and, once that
// queue is used up, takes what is left in the others.
//
// Line mode (a few trajectories: fewer tiles than keep 256 CUs busy, each as
// long as the whole context): the key blocks of all (KV head, tile) pairs form
// one line, cut into up to kShares equal shares, one per workgroup, so that
// every CU gets the same number of key blocks however few tiles there are. A
// share ends inside a tile as a rule; the pieces of a tile that more than one
// share touches are merged by append_merge_kernel. Shares of one XCD are
// adjacent on the line (with 8 KV heads, one head per XCD). What bounds a call
// in this mode is the key loop itself, evenly spread; a whole tile per CU was
// bound by the longest tile's chain of key blocks with most CUs idle. Measured
// (Hq 32, Hkv 8, queue mode -> line mode): 2 rows of 64..512 new tokens over
// 2k..24k keys 532 -> 205 us, 1 row of 200 over 16k 421 -> 97 us, 1 row of 10
// over 30k 746 -> 54 us, 1 row of 30 over 3k 96 -> 35 us.
// Where each way is used: line mode when a share plus 16 key blocks (what
// writing and merging the partial results costs a share, about 30 us) is
// shorter than the longest tile, which bounds queue mode from below. Both
// sides of the line: a first prompt of 2,000 tokens (256 tiles of 1 to 32
// blocks, 16.5 blocks a share) takes 81 us queued and 107 us as a line; 8 rows
// over 2 KV heads 692 us queued and 575 us as a line. With far more tiles than
// CUs the line loses the sharing of K/V in the XCD's L2: 64 mixed rows 7.0 ms
// queued and 8.0 ms as a line. Decode rows beside the append rows do not enter the
// rule (a mixed call's append rows get the bits of the append call): all shares come
// before the decode splits, where queued tiles run beside them. That gains the more
// the longer the tiles (32 decode rows of 16k with 2 rows of 256 over 12k 794 -> 574
// us) and loses 1 to 2 % where decode is most of the call (256 such rows with 1 row of
// 64 over 16k 2,686 -> 2,717 us); shares spread over the decode splits were slower.
//
// Decode splits (row, split, KV head) are queued per XCD in both modes, row by
// row. In each queue the workgroups take the next entry of one merged order
// from a device counter. The merged order places the decode splits at even
// spacing among the queued append tiles, so that a few CUs stream KV pages for
// decode (bound by HBM) while the rest run the append tiles' matrix products
// (bound by the matrix cores). Entry j of a queue's merged order (n entries,
// nd of them decode splits) is decode split floor(j nd / n) when
// floor((j + 1) nd / n) > floor(j nd / n), else append tile
// j - floor(j nd / n).
// A decode split is computed as by the decode split kernel but with 8 waves;
// the decode combine follows as in plain decode. Results do not depend on
// the order in which entries are taken, and how the append tiles are cut
// depends on the append rows' lengths and places in the call alone.
#include <atomic>

#include "ra_append_tile.h"
#include "ra_decode_split.h"
#include "ra_internal.h"
#include "ra_page_write.h"

namespace ra {
namespace {

constexpr int kMixWaves = 8;
constexpr int kMixThreads = kMixWaves * kWave;
static_assert(kMixThreads == atile::kThreads, "append tiles take the whole workgroup");
constexpr int kPlanThreads = 1024;
constexpr int kPlanWaves = kPlanThreads / kWave;
constexpr int kOwnTiles = 4;         // tiles up to which a row is listed by one thread
constexpr int kCostBuckets = 4096;   // key-block counts above this share the last bucket
constexpr int kHeadBits = 8;         // KV heads of a call: at most 1 << kHeadBits
constexpr int kQueues = 8;           // one work queue per XCD
constexpr int kShares = 256;         // line mode: most shares (one per CU of an MI355X)
constexpr int kMinShare = 4;         // line mode: fewest key blocks a share is cut to. More
                                     // pieces cost merging, fewer leave compute units idle: 2, 4
                                     // and 8 measure 39, 35 and 33 us at 1 row of 30 over 3k
                                     // keys and 44, 51 and 53 us at 1 row of 200 over 1k; no
                                     // value is best at both
constexpr int kLineCost = 16;        // line mode: key blocks its partial results cost a share
constexpr int64_t kMaxLine = 1 << 28;   // line mode: most key blocks (int32 positions)

// header words: per queue q [q] next entry
enum { kHdrTiles = 8, kHdrSplits, kHdrShares, kHdrShare, kHdrHead };
// kHdrTiles    append tiles (row, query block)
// kHdrSplits   decode splits (row, split)
// kHdrShares   line mode: number of shares (0: queue mode)
// kHdrShare    line mode: key blocks per share
// kHdrHead     line mode: key blocks of one KV head's tiles

struct MixedArgs {
  atile::AppendArgs ap;
  dsplit::DecodeArgs de;
  atile::AppendTile *tiles;   // append tiles, in the order they are taken
  int32_t *tile_start;   // line mode: key blocks of one head before each tile
  int32_t *split_start;  // decode splits before each decode row
  int32_t *order;        // append rows, longest chunk end first
  int32_t *header;
  int4 *cut;             // [kShares] tile whose first piece ends share w: {row, query block,
                         // KV head, pieces} (pieces 0: none)
  atile::PartialOut part;   // line mode: slots 2w (a piece that continues a tile) and
                            // 2w + 1 (a tile's first piece) of share w
  int32_t B_append;
};

// Exclusive prefix sum of v over the kPlanThreads threads of the workgroup;
// *total receives the sum of all. Every thread calls it. s: kPlanWaves ints.
__device__ int block_exclusive_scan(int v, int *s, int *total) {
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  int incl = v;
#pragma unroll
  for (int off = 1; off < kWave; off *= 2) {
    const int t = __shfl_up(incl, off);
    if (lane >= off) incl += t;
  }
  if (lane == kWave - 1) s[wave] = incl;
  __syncthreads();
  int before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < kPlanWaves; ++w) {
    const int t = s[w];
    before += w < wave ? t : 0;
    all += t;
  }
  *total = all;
  __syncthreads();   // s may be reused by the caller
  return before + incl - v;
}

// KV heads g = q, q + 8, ... below hkv go to queue q.
__device__ __forceinline__ int heads_of_queue(int hkv, int q) {
  return q < hkv ? (hkv - 1 - q) / kQueues + 1 : 0;
}

// Query blocks of row b with work (0 for an empty row).
__device__ __forceinline__ int row_qblocks(const atile::AppendArgs &ap, const atile::AppendRow &r) {
  if (r.T <= 0 || r.ctx < 0) return 0;
  return (r.T + ap.q_per_block - 1) / ap.q_per_block;
}

// Key blocks of the first nq tiles of a row (all of them).
__device__ __forceinline__ int64_t row_blocks(const atile::AppendArgs &ap, const atile::AppendRow &r,
                                              int nq) {
  int64_t sum = 0;
  for (int qb = 0; qb < nq; ++qb) sum += atile::append_tile_blocks(ap, r, qb);
  return sum;
}

// Workgroup 0 plans. With the page write fused in, every other workgroup writes
// four (page, kFusedHeads KV heads) units of the chunks' K/V meanwhile; the attention kernel after this one
// reads them from the pool.
constexpr int kFusedHeads = 2;   // KV heads of a write unit here (LDS for 2 workgroups per CU)
__global__ __launch_bounds__(kPlanThreads) void mixed_plan_kernel(MixedArgs m, pwrite::WriteArgs w,
                                                                  int64_t write_units) {
  if (blockIdx.x > 0) {
    constexpr int kPer = kPlanThreads / pwrite::kItemThreads;
    __shared__ uint16_t sv[kPer][kFusedHeads][kPage][pwrite::kVPitch];
    const int part = threadIdx.x / pwrite::kItemThreads, t = threadIdx.x % pwrite::kItemThreads;
    const int64_t unit = (int64_t)(blockIdx.x - 1) * kPer + part;
    const int groups = (w.hkv + kFusedHeads - 1) / kFusedHeads;
    const int item = (int)(unit / groups), g0 = (int)(unit - (int64_t)item * groups) * kFusedHeads;
    pwrite::WriteItem it;
    it.active = false;
    if (unit < write_units) it = pwrite::item_page(w, m.B_append, item);
    if (w.fp8 && w.cos_sin)
      pwrite::write_heads<true, true, kFusedHeads>(w, it, g0, t, sv[part]);
    else if (w.fp8)
      pwrite::write_heads<true, false, kFusedHeads>(w, it, g0, t, sv[part]);
    else if (w.cos_sin)
      pwrite::write_heads<false, true, kFusedHeads>(w, it, g0, t, sv[part]);
    else
      pwrite::write_heads<false, false, kFusedHeads>(w, it, g0, t, sv[part]);
    return;
  }
  __shared__ int count[kCostBuckets];   // rows per key-block count, then write cursors
  __shared__ int s_scan[kPlanWaves];
  __shared__ int s_longest;
  __shared__ unsigned long long s_blocks;
  __shared__ int s_row[kPlanThreads][2];   // a chunk of ranked rows: tiles and key blocks before
  __shared__ int s_long[kPlanThreads], s_num_long;   // rows of the chunk that waves list
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1), wave = tid / kWave;
  const int hkv_a = m.ap.hkv;
  for (int c = tid; c < kCostBuckets; c += kPlanThreads) count[c] = 0;
  if (tid == 0) s_longest = 0, s_blocks = 0;
  if (tid < kQueues) m.header[tid] = 0;
  __syncthreads();

  // ---- append rows, by the key blocks of their longest (last) tile, longest
  // first; the key blocks of all tiles and the longest tile
  for (int b = tid; b < m.B_append; b += kPlanThreads) {
    const atile::AppendRow r = atile::append_row(m.ap, b);
    const int nq = row_qblocks(m.ap, r);
    if (nq == 0) continue;
    const int nb = atile::append_tile_blocks(m.ap, r, nq - 1);
    atomicAdd(&count[min(nb, kCostBuckets) - 1], 1);
    atomicMax(&s_longest, nb);
    atomicAdd(&s_blocks, (unsigned long long)row_blocks(m.ap, r, nq));
  }
  __syncthreads();
  const int64_t head_blocks = (int64_t)s_blocks, line = head_blocks * hkv_a;
  constexpr int kPer = kCostBuckets / kPlanThreads;
  int own[kPer], sum = 0;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    own[k] = count[kCostBuckets - 1 - (kPer * tid + k)];
    sum += own[k];
  }
  int n_rows;
  int cursor = block_exclusive_scan(sum, s_scan, &n_rows);
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    count[kCostBuckets - 1 - (kPer * tid + k)] = cursor;
    cursor += own[k];
  }
  __syncthreads();
  // ---- line mode: when a share and what its partial results cost take less
  // than the longest tile
  int shares = 0, share = 0;
  if (line <= kMaxLine && line < (int64_t)kShares * (s_longest - kLineCost)) {
    shares = (int)min((int64_t)kShares, (line + kMinShare - 1) / kMinShare);
    share = (int)((line + shares - 1) / shares);
    shares = (int)((line + share - 1) / share);
  }

  // ---- places: the rows of a bucket take them in turn. In line mode, where a row's
  // place decides how its tiles are cut, rows of one bucket are placed by row number
  // (a thread counts those before it among the 1,024 of its round); in queue mode the
  // order only says who starts first.
  if (shares) {
    int *const s_bucket = &s_row[0][0];
    for (int b0 = 0; b0 < m.B_append; b0 += kPlanThreads) {
      const int b = b0 + tid;
      int bucket = -1;
      if (b < m.B_append) {
        const atile::AppendRow r = atile::append_row(m.ap, b);
        const int nq = row_qblocks(m.ap, r);
        if (nq > 0) bucket = min(atile::append_tile_blocks(m.ap, r, nq - 1), kCostBuckets) - 1;
      }
      s_bucket[tid] = bucket;
      __syncthreads();
      if (bucket >= 0) {
        int before = 0;
        for (int i = 0; i < tid; ++i) before += s_bucket[i] == bucket;
        m.order[count[bucket] + before] = b;
      }
      __syncthreads();
      if (bucket >= 0) atomicAdd(&count[bucket], 1);
      __syncthreads();
    }
  } else {
    for (int b = tid; b < m.B_append; b += kPlanThreads) {
      const atile::AppendRow r = atile::append_row(m.ap, b);
      const int nq = row_qblocks(m.ap, r);
      if (nq == 0) continue;
      const int nb = atile::append_tile_blocks(m.ap, r, nq - 1);
      m.order[atomicAdd(&count[min(nb, kCostBuckets) - 1], 1)] = b;
    }
    __syncthreads();
  }

  // ---- tiles: rows in the order above, each row's query blocks last first; a thread
  // lists a row of few tiles, a wave a row of many (a call of 2,000 rows of one tile: 175 us,
  // 255 us with a wave for every row)
  int done_tiles = 0, done_blocks = 0;   // of the rows ranked before this chunk
  for (int k0 = 0; k0 < n_rows; k0 += kPlanThreads) {
    const int k = k0 + tid, b = k < n_rows ? m.order[k] : 0;
    atile::AppendRow r = {0, 0, 0};
    int nq = 0, nb = 0;
    if (k < n_rows) {
      r = atile::append_row(m.ap, b);
      nq = row_qblocks(m.ap, r);
      if (shares) nb = (int)row_blocks(m.ap, r, nq);
    }
    if (tid == 0) s_num_long = 0;
    int chunk_tiles, chunk_blocks = 0, blocks = 0;
    const int first = done_tiles + block_exclusive_scan(nq, s_scan, &chunk_tiles);
    if (shares) blocks = done_blocks + block_exclusive_scan(nb, s_scan, &chunk_blocks);
    if (nq > kOwnTiles) {
      s_row[tid][0] = first, s_row[tid][1] = blocks;
      s_long[atomicAdd(&s_num_long, 1)] = tid;
    } else {
      for (int i = 0; i < nq; ++i) {
        m.tiles[first + i] = atile::make_tile(m.ap, r, b, nq - 1 - i);
        if (shares) m.tile_start[first + i] = blocks;
        blocks += atile::append_tile_blocks(m.ap, r, nq - 1 - i);
      }
    }
    __syncthreads();
    for (int j = wave; j < s_num_long; j += kPlanWaves) {
      const int kk = s_long[j], row = m.order[k0 + kk];
      const atile::AppendRow rr = atile::append_row(m.ap, row);
      const int row_nq = row_qblocks(m.ap, rr), row_first = s_row[kk][0];
      int before = s_row[kk][1];
      for (int i0 = 0; i0 < row_nq; i0 += kWave) {
        const int i = i0 + lane, qb = row_nq - 1 - i;
        if (i < row_nq) m.tiles[row_first + i] = atile::make_tile(m.ap, rr, row, qb);
        if (shares) {
          const int n = i < row_nq ? atile::append_tile_blocks(m.ap, rr, qb) : 0;
          int incl = n;
#pragma unroll
          for (int off = 1; off < kWave; off *= 2) {
            const int t = __shfl_up(incl, off);
            if (lane >= off) incl += t;
          }
          if (i < row_nq) m.tile_start[row_first + i] = before + incl - n;
          before += __shfl(incl, kWave - 1);
        }
      }
    }
    done_tiles += chunk_tiles;
    done_blocks += chunk_blocks;
    __syncthreads();   // s_row and s_long are written again
  }

  // ---- decode splits before each row
  const int S = m.de.split_tokens;
  int total_ns = 0;
  for (int r0 = 0; r0 < m.de.B; r0 += kPlanThreads) {
    const int b = r0 + tid;
    const int ns = b < m.de.B ? (dsplit::row_len(m.de, b) + S - 1) / S : 0;
    int chunk;
    const int before = total_ns + block_exclusive_scan(ns, s_scan, &chunk);
    if (b < m.de.B) m.split_start[b] = before;
    total_ns += chunk;
  }
  if (tid < kShares) m.cut[tid] = make_int4(0, 0, 0, 0);
  if (tid == 0) {
    m.header[kHdrTiles] = done_tiles;
    m.header[kHdrSplits] = total_ns;
    m.header[kHdrShares] = shares;
    m.header[kHdrShare] = share;
    m.header[kHdrHead] = (int)head_blocks;   // read in line mode only (it then fits)
  }
}

// Line mode: the share of this workgroup, or -1. Workgroups are placed on the
// XCDs round robin; adjacent shares go to one XCD's workgroups.
__device__ __forceinline__ int share_of_workgroup(int shares) {
  const int per = (shares + kQueues - 1) / kQueues;
  const int k = (int)blockIdx.x / kQueues, w = ((int)blockIdx.x % kQueues) * per + k;
  return k < per && w < shares ? w : -1;
}

__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

// A tile of the list, in scalar registers.
__device__ __forceinline__ atile::AppendTile load_tile(const MixedArgs &m, int i) {
  const u32x4 *p = reinterpret_cast<const u32x4 *>(m.tiles + i);
  const u32x4 lo = p[0], hi = p[1];
  return atile::AppendTile{uniform(lo[0]), uniform(lo[1]), uniform(lo[2]), uniform(lo[3]),
                           uniform(hi[0]), uniform(hi[1]), {0, 0}};
}

template <typename T>
__device__ __forceinline__ void global_ptr(T *&p) {
  p = (T *)(__attribute__((address_space(1))) T *)(uintptr_t)p;
}

// The kernel's arguments, read again from the kernel argument segment where
// they are used: kept in scalar registers through the entry loop, the decode
// and append arguments together overflow them.
__device__ __forceinline__ MixedArgs reload_args() {
  typedef const __attribute__((address_space(4))) uint64_t *ConstWords;
  ConstWords p = (ConstWords)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  static_assert(sizeof(MixedArgs) % 8 == 0, "whole words");
  uint64_t w[sizeof(MixedArgs) / 8];
#pragma unroll
  for (size_t i = 0; i < sizeof(MixedArgs) / 8; ++i) w[i] = p[i];
  MixedArgs m = __builtin_bit_cast(MixedArgs, w);
  // every pointer is to global memory (the compiler knows so of kernel
  // arguments only; it would otherwise take the slower flat accesses)
  global_ptr(m.ap.q), global_ptr(m.ap.k_pool), global_ptr(m.ap.v_pool);
  global_ptr(m.ap.block_table), global_ptr(m.ap.cu_q), global_ptr(m.ap.ctx_lens);
  global_ptr(m.ap.out), global_ptr(m.ap.lse), global_ptr(m.ap.cos_sin);
  global_ptr(m.de.q), global_ptr(m.de.k_pool), global_ptr(m.de.v_pool);
  global_ptr(m.de.block_table), global_ptr(m.de.kv_lens), global_ptr(m.de.group_start);
  global_ptr(m.de.prefix_len), global_ptr(m.de.ws_o), global_ptr(m.de.ws_m), global_ptr(m.de.ws_l);
  global_ptr(m.tiles), global_ptr(m.tile_start), global_ptr(m.split_start), global_ptr(m.order);
  global_ptr(m.header), global_ptr(m.cut), global_ptr(m.part.o), global_ptr(m.part.ml);
  return m;
}

// kDecode: the call has decode rows (otherwise every entry is an append tile).
// kFp8: the pools hold E4M3 codes. kRope: the append rows' q is rotated at its
// position (append-only calls). kDecodeTiles: 16-column tiles of a decode
// split (2 for groups of 17 to 32 query heads).
template <bool kPosScale, bool kDecode, bool kFp8, bool kRope = false, int kDecodeTiles = 1>
__global__ __launch_bounds__(kMixThreads, 1) void mixed_kernel(MixedArgs args) {
  __shared__ union {
    atile::AppendLds ap;
    dsplit::DecodeLds<kDecodeTiles, kMixWaves> de;
  } lds;
  // What a workgroup keeps between entries lives in LDS (the append tile leaves
  // no registers for it), twice: thread 0 writes what follows an entry before
  // the entry's end, when other waves may still be reading what it was.
  struct State {
    int ticket;    // entry of queue `queue` (-1: none taken yet)
    int queue;     // queues used up: first this XCD's queue, then the others
    int pos, end;  // what is left of the workgroup's share of the line
    int tile;      // the tile at pos
  };
  __shared__ State s_state[2];
  __shared__ int s_header[8];
  enum { kTiles, kSplits, kShareCount, kShare, kHead };   // m.header[8 + ...]
  if (threadIdx.x < 8) s_header[threadIdx.x] = args.header[8 + threadIdx.x];
  __syncthreads();
  if (threadIdx.x < kWave) {
    const MixedArgs &m = args;
    State st = {-1, 0, 0, 0, 0};
    const int w = share_of_workgroup(s_header[kShareCount]);
    if (w >= 0) {
      const int64_t line = (int64_t)s_header[kHead] * m.ap.hkv, share = s_header[kShare];
      st.pos = (int)(w * share);
      st.end = (int)min(line, (w + 1) * share);
      st.tile = wave_search(s_header[kTiles], st.pos % s_header[kHead],
                            [&](int i) { return m.tile_start[i]; });
    }
    if (threadIdx.x == 0) s_state[0] = st;
  }
  for (int cur = 0;; cur ^= 1) {
    __syncthreads();   // the previous entry is done with LDS; s_state[cur] is there
    const MixedArgs m = reload_args();
    State st = {uniform(s_state[cur].ticket), uniform(s_state[cur].queue),
                uniform(s_state[cur].pos), uniform(s_state[cur].end),
                uniform(s_state[cur].tile)};
    const int nt = s_header[kShareCount] ? 0 : uniform(s_header[kTiles]);
    const int ns = kDecode ? uniform(s_header[kSplits]) : 0;
    int index, head, kb0 = 0, kb1 = 0, slot = -1;
    bool decode = false;
    if (st.pos < st.end) {   // a piece of the line
      const int head_blocks = uniform(s_header[kHead]);
      head = st.pos / head_blocks;
      index = st.tile;
      kb0 = st.pos - head * head_blocks - uniform(m.tile_start[index]);
    } else {   // the next entry of the queues
      int q, ha, hd;
      int64_t n;
      for (;;) {
        q = ((int)blockIdx.x + st.queue) % kQueues;
        ha = heads_of_queue(m.ap.hkv, q), hd = heads_of_queue(m.de.hkv, q);
        n = (int64_t)nt * ha + (int64_t)ns * hd;
        if (st.ticket >= 0 && st.ticket < n) break;
        // none, or past this queue's end: a ticket of the next one with work
        if (st.ticket >= 0 || n == 0) {
          if (++st.queue >= kQueues) return;
          st.ticket = -1;
          continue;
        }
        __syncthreads();
        if (threadIdx.x == 0) s_state[cur].ticket = atomicAdd(&m.header[q], 1);
        __syncthreads();
        st.ticket = uniform(s_state[cur].ticket);
      }
      const int64_t nd = (int64_t)ns * hd;
      const int j = st.ticket, dj = (int)(j * nd / n);
      decode = kDecode && (int)((j + 1) * nd / n) > dj;
      if (decode) {
        head = q + kQueues * (dj % hd);
        index = dj / hd;
      } else {
        head = q + kQueues * ((j - dj) % ha);
        index = (j - dj) / ha;
      }
    }
    if (decode) {
      const int row = wave_search(m.de.B, index, [&](int i) { return m.split_start[i]; });
      dsplit::decode_split<kDecodeTiles, false, kMixWaves, kFp8>(
          m.de, head, index - uniform(m.split_start[row]), row, lds.de);
      if (threadIdx.x == 0)
        s_state[cur ^ 1] = {atomicAdd(&m.header[((int)blockIdx.x + st.queue) % kQueues], 1),
                            st.queue, 0, 0, 0};
    } else {
      const atile::AppendTile tile = load_tile(m, index);
      kb1 = tile.blocks;
      const bool line = st.pos < st.end;
      if (line) {   // a piece that does not start or end its tile is partial
        const int w = share_of_workgroup(uniform(s_header[kShareCount]));
        kb1 = min(kb1, kb0 + st.end - st.pos);
        slot = kb0 > 0 ? 2 * w : kb1 < tile.blocks ? 2 * w + 1 : -1;
        if (kb0 == 0 && kb1 < tile.blocks && threadIdx.x == 0)
          // the tile ends in share (st.pos + tile.blocks - 1) / share
          m.cut[w] = make_int4(tile.row, tile.qblk, head,
                               (st.pos + tile.blocks - 1) / s_header[kShare] - w + 1);
      }
      // the ticket of the next entry, taken only near the end of this one: a
      // ticket held through a long tile would leave other CUs idle at the end
      auto issue = [&]() __attribute__((always_inline)) {
        return line || threadIdx.x != 0
                   ? 0
                   : atomicAdd(&m.header[((int)blockIdx.x + st.queue) % kQueues], 1);
      };
      auto commit = [&](int ticket) __attribute__((always_inline)) {
        if (threadIdx.x != 0) return;
        s_state[cur ^ 1] = line ? State{-1, 0, st.pos + kb1 - kb0, st.end,
                                        index + 1 < s_header[kTiles] ? index + 1 : 0}
                                : State{ticket, st.queue, 0, 0, 0};
      };
      atile::append_tile<kPosScale, kFp8, kRope>(m.ap, tile, head, kb0, kb1, slot, m.part, lds.ap,
                                                 issue, commit);
    }
  }
}

// Merge of the pieces of the cut tiles (line mode): of the tile that share w starts and
// does not end, pieces 2w + 1, 2(w + 1), ..., in this order. The cut tiles' query rows, 32 at
// a time (32 lanes each, with four dims of a row), are dealt to kMergeGroups workgroups, few
// enough that a call in queue mode, which launches them for nothing, loses 2 us (a
// workgroup for every 8 rows of every share: 3.4 us); 2 rows of 64..512 new tokens over
// 2k..24k keys take 195 us a call with these, 204 us with those.
constexpr int kMergeThreads = 1024;
constexpr int kMergeGroups = 512;
constexpr int kMergeRows = kMergeThreads / 32;
constexpr int kMergeParts = atile::kRowsPerGroup / kMergeRows;
__global__ __launch_bounds__(kMergeThreads) void append_merge_kernel(MixedArgs m) {
  if (m.header[kHdrShares] == 0) return;
  // the shares with a cut tile, in order
  __shared__ int s_cut[kShares];
  __shared__ int s_count[kShares / kWave];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const bool is_cut = tid < kShares && m.cut[tid].w > 0;
  const unsigned long long cut_lanes = __ballot(is_cut);
  if (tid < kShares && lane == 0) s_count[wave] = (int)__popcll(cut_lanes);
  __syncthreads();
  int before = 0, cuts = 0;
  for (int v = 0; v < kShares / kWave; ++v) {
    before += v < wave ? s_count[v] : 0;
    cuts += s_count[v];
  }
  if (is_cut) s_cut[before + (int)__popcll(cut_lanes & ((1ull << lane) - 1))] = tid;
  __syncthreads();

  const int G = m.ap.group, d = (tid & 31) * 4;
  for (int item = blockIdx.x; item < cuts * kMergeParts; item += kMergeGroups) {
    const int w = s_cut[item / kMergeParts];
    const int4 cut = m.cut[w];
    const atile::AppendRow r = atile::append_row(m.ap, cut.x);
    const int i0 = cut.y * m.ap.q_per_block;
    const int rows = min(r.T - i0, m.ap.q_per_block) * G;   // query rows of the tile
    const int row = item % kMergeParts * kMergeRows + tid / 32;
    if (row >= rows) continue;
    auto slot = [&](int p) { return (2 * (w + p) + (p == 0)) * (size_t)m.part.rows + row; };
    // eight pieces' loads in flight together
    constexpr int kBatch = 8;
    float M = -INFINITY;
    for (int p0 = 0; p0 < cut.w; p0 += kBatch) {
      float mv[kBatch];
#pragma unroll
      for (int j = 0; j < kBatch; ++j) mv[j] = m.part.ml[slot(min(p0 + j, cut.w - 1))].x;
#pragma unroll
      for (int j = 0; j < kBatch; ++j) M = fmaxf(M, mv[j]);
    }
    const float M_use = M == -INFINITY ? 0.f : M;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    float l = 0.f;
    for (int p0 = 0; p0 < cut.w; p0 += kBatch) {
      float f[kBatch], lp[kBatch];
      f32x4 o[kBatch];
#pragma unroll
      for (int j = 0; j < kBatch; ++j) {
        const size_t s = slot(min(p0 + j, cut.w - 1));
        const float2 ml = m.part.ml[s];
        o[j] = *reinterpret_cast<const f32x4 *>(&m.part.o[s * kHeadDim + d]);
        f[j] = fast_exp2(ml.x - M_use);
        lp[j] = ml.y;
      }
#pragma unroll
      for (int j = 0; j < kBatch; ++j)
        if (p0 + j < cut.w) {
          acc += f[j] * o[j];
          l += f[j] * lp[j];
        }
    }
    const int qi = row / G;
    const size_t out = (size_t)(r.cu0 + i0 + qi) * m.ap.hq + (size_t)cut.z * G + (row - qi * G);
    const float inv = m.ap.v_scale / l;
    *reinterpret_cast<f32x4 *>(&m.ap.out[out * kHeadDim + d]) = acc * inv;
    if (m.ap.lse && d == 0) m.ap.lse[out] = (M + __log2f(l)) * kLn2;
  }
}

constexpr size_t kAlign = 256;
size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

// Compute units of the current device, queried once per device (a device's
// count never changes; racing first calls store the same value).
constexpr int kMaxDevices = 64;
std::atomic<int> g_cus[kMaxDevices];
hipError_t device_cus(int *cus) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices)
    return hipDeviceGetAttribute(cus, hipDeviceAttributeMultiprocessorCount, dev);
  int n = g_cus[dev].load(std::memory_order_relaxed);
  if (n <= 0) {
    if ((e = hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess)
      return e;
    g_cus[dev].store(n, std::memory_order_relaxed);
  }
  *cus = n;
  return hipSuccess;
}

}  // namespace

MixedLayout mixed_layout(int32_t B_decode, int32_t B_append, int32_t hq, int32_t hkv_decode,
                         int32_t hkv_append, int32_t max_kv_len_decode, int32_t max_q_len) {
  MixedLayout l;
  l.plan = decode_plan(B_decode > 0 ? B_decode : 1, hkv_decode, max_kv_len_decode);
  const int32_t qpb = atile::kRowsPerGroup / (hq / hkv_append);
  l.qblocks = max_q_len > 0 ? (int32_t)(((int64_t)max_q_len + qpb - 1) / qpb) : 0;
  l.max_tiles = (int64_t)B_append * l.qblocks * hkv_append;
  l.max_splits = (int64_t)B_decode * l.plan.max_splits * hkv_decode;
  // the header, the share cuts and the append row order, then the lists (the tile list
  // no smaller than the 8 bytes per tile and KV head that this size has always held,
  // which what callers compare it with may count on) and the partial results: two
  // pieces a share, of the query rows that the fullest tile can have (17 MB for chunks
  // of up to 16 tokens and 4 heads a KV head, 68 MB from 64 tokens)
  l.order_offset = kAlign + align_up(kShares * sizeof(int4));
  l.tiles_offset = l.order_offset + align_up((size_t)(B_append > 0 ? B_append : 0) * sizeof(int32_t));
  const size_t tiles = (size_t)(l.max_tiles / hkv_append);
  const size_t per_head = (size_t)l.max_tiles * sizeof(int2);
  const size_t listed = tiles * sizeof(atile::AppendTile);
  l.starts_offset = l.tiles_offset + align_up(per_head > listed ? per_head : listed);
  l.splits_offset =
      l.starts_offset + align_up(tiles * sizeof(int32_t));
  l.partials_offset =
      l.splits_offset + align_up((size_t)(B_decode > 0 ? B_decode : 0) * sizeof(int32_t));
  l.pieces_offset = align_up(l.partials_offset +
                             (B_decode > 0 ? decode_workspace_bytes(B_decode, hq, l.plan) : 0));
  l.piece_rows = (max_q_len < qpb ? max_q_len : qpb) * (hq / hkv_append);
  const size_t piece_rows = l.max_tiles > 0 ? (size_t)2 * kShares * l.piece_rows : 0;
  l.bytes = l.pieces_offset + piece_rows * (kHeadDim * sizeof(float) + sizeof(float2));
  return l;
}

int32_t mixed_hkv_limit() { return 1 << kHeadBits; }

namespace {
constexpr int64_t kUnitsPer = kPlanThreads / pwrite::kItemThreads;
int64_t fused_write_units(int32_t B, int32_t total_q, int32_t hkv) {
  return pwrite::write_items(B, total_q) * ((hkv + kFusedHeads - 1) / kFusedHeads);
}
}  // namespace

int64_t fused_write_blocks(int32_t B, int32_t total_q, int32_t hkv) {
  return (fused_write_units(B, total_q, hkv) + kUnitsPer - 1) / kUnitsPer;
}

hipError_t launch_mixed(const uint16_t *q_decode, const PagedKV &kv_decode,
                        const int32_t *kv_lens, int32_t B_decode, int32_t max_kv_len_decode,
                        float *out_decode, float *lse_decode, const uint16_t *q_append,
                        const int32_t *cu_q, const int32_t *ctx_lens, const PagedKV &kv_append,
                        int32_t B_append, int32_t total_q, int32_t max_q_len,
                        int32_t max_kv_len_append, float *out_append, float *lse_append,
                        int32_t hq, float scale, void *workspace, const MixedLayout &layout,
                        hipStream_t stream, const uint16_t *k_new, const uint16_t *v_new,
                        const float *cos_sin, int32_t rope_rows) {
  char *ws = static_cast<char *>(workspace);
  MixedArgs m;
  m.ap = atile::make_append_args(q_append, cu_q, ctx_lens, kv_append, hq, total_q, max_q_len,
                                 max_kv_len_append, scale, out_append, lse_append);
  m.ap.cos_sin = cos_sin;   // q of the append rows rotated at their positions (or not)
  m.ap.rope_rows = rope_rows;
  m.de = dsplit::make_decode_args(q_decode, kv_decode, kv_lens, B_decode, hq,
                                  max_kv_len_decode, scale, ws + layout.partials_offset,
                                  layout.plan.max_splits, layout.plan);
  m.header = reinterpret_cast<int32_t *>(ws);
  m.cut = reinterpret_cast<int4 *>(ws + kAlign);
  m.order = reinterpret_cast<int32_t *>(ws + layout.order_offset);
  m.tiles = reinterpret_cast<atile::AppendTile *>(ws + layout.tiles_offset);
  m.tile_start = reinterpret_cast<int32_t *>(ws + layout.starts_offset);
  m.split_start = reinterpret_cast<int32_t *>(ws + layout.splits_offset);
  m.part.o = reinterpret_cast<float *>(ws + layout.pieces_offset);
  m.part.rows = layout.piece_rows;
  m.part.ml = reinterpret_cast<float2 *>(
      m.part.o + (size_t)2 * kShares * layout.piece_rows * kHeadDim);
  m.B_append = B_append;

  // the fused page write (append rows only): the chunks' tokens at ctx_lens
  const pwrite::WriteArgs w = pwrite::write_args(k_new, v_new, cu_q, ctx_lens, kv_append, total_q,
                                                 max_q_len, max_kv_len_append, cos_sin, rope_rows);
  const int64_t write_units = k_new ? fused_write_units(B_append, total_q, kv_append.hkv) : 0;
  const int64_t write_blocks = (write_units + kUnitsPer - 1) / kUnitsPer;
  hipLaunchKernelGGL(mixed_plan_kernel, dim3((unsigned)(1 + write_blocks)), dim3(kPlanThreads), 0,
                     stream, m, w, write_units);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // One workgroup per CU: the kernel's registers allow one 8-wave
  // workgroup per CU, and every workgroup runs until the entries run out.
  int cus = 0;
  if ((e = device_cus(&cus)) != hipSuccess) return e;
  // A line of few tiles is cut into up to kShares shares of kMinShare key
  // blocks or more, and every share has its own workgroup.
  const int64_t tile_blocks = ((int64_t)max_kv_len_append + atile::kBlock - 1) / atile::kBlock;
  const int64_t cuts = B_append > 0 ? layout.max_tiles * (tile_blocks / kMinShare + 1) : 0;
  const int64_t line_wgs =
      ((cuts < kShares ? cuts : kShares) + kQueues - 1) / kQueues * kQueues;
  const int64_t entries = layout.max_tiles + layout.max_splits;
  int64_t wgs = entries < cus ? (entries > 0 ? entries : 1) : cus;
  if (wgs < line_wgs) wgs = line_wgs;
  const unsigned grid = (unsigned)wgs;
  const dim3 g(grid), b(kMixThreads);
  const bool pos = m.ap.scale_log2 > 0.f || B_append == 0;
  const bool fp8 = kv_decode.fp8 || kv_append.fp8;   // the ABI layer allows one element type
  // rotated queries come only with append-only calls (the fused rotated write)
  if (cos_sin && B_decode > 0) return hipErrorInvalidValue;
  if (B_decode > 0 && m.de.group > 16) {   // two-tile decode splits
    const int v2 = (pos ? 2 : 0) | (fp8 ? 1 : 0);
    if (v2 == 0) hipLaunchKernelGGL((mixed_kernel<false, true, false, false, 2>), g, b, 0, stream, m);
    if (v2 == 1) hipLaunchKernelGGL((mixed_kernel<false, true, true, false, 2>), g, b, 0, stream, m);
    if (v2 == 2) hipLaunchKernelGGL((mixed_kernel<true, true, false, false, 2>), g, b, 0, stream, m);
    if (v2 == 3) hipLaunchKernelGGL((mixed_kernel<true, true, true, false, 2>), g, b, 0, stream, m);
  } else {
    const int variant = (cos_sin ? 8 : 0) | (pos ? 4 : 0) | (B_decode > 0 ? 2 : 0) | (fp8 ? 1 : 0);
    switch (variant) {
#define RA_MIXED_CASE(V, P, D, F, R)                                                  \
  case V:                                                                             \
    hipLaunchKernelGGL((mixed_kernel<P, D, F, R>), g, b, 0, stream, m);               \
    break;
      RA_MIXED_CASE(0, false, false, false, false)
      RA_MIXED_CASE(1, false, false, true, false)
      RA_MIXED_CASE(2, false, true, false, false)
      RA_MIXED_CASE(3, false, true, true, false)
      RA_MIXED_CASE(4, true, false, false, false)
      RA_MIXED_CASE(5, true, false, true, false)
      RA_MIXED_CASE(6, true, true, false, false)
      RA_MIXED_CASE(7, true, true, true, false)
      RA_MIXED_CASE(8, false, false, false, true)
      RA_MIXED_CASE(9, false, false, true, true)
      RA_MIXED_CASE(12, true, false, false, true)
      RA_MIXED_CASE(13, true, false, true, true)
#undef RA_MIXED_CASE
    }
  }
  if ((e = hipGetLastError()) != hipSuccess) return e;
  // (line mode needs a tile of more than kLineCost key blocks)
  if (B_append > 0 && tile_blocks > kLineCost) {
    hipLaunchKernelGGL(append_merge_kernel, dim3(kMergeGroups), dim3(kMergeThreads), 0,
                       stream, m);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if (B_decode == 0) return hipSuccess;
  dsplit::launch_combine(m.de, B_decode, out_decode, lse_decode, stream);
  return hipGetLastError();
}

}  // namespace ra
