// Per-token log-probabilities under an LM head, fused: logits, log-sum-exp and
// the gather of the emitted token's logit, without writing the logits.
//
// For token n (hidden state h[n], emitted token t[n]) and the LM-head matrix
// W [V][D]: z_v = scale * <h[n], W[v]>, lse = ln sum_v exp z_v, and
// logp = z_t - lse.
//
// Which kernel writes the partials (one (max, sum) per token and vocabulary
// chunk), by batch size and layout of W; times at V = 151,936, D = 4,096 with
// the alternative beside it:
// - N <= 128, packed: logprob_partial_kernel. 4 waves per 128-row chunk, W
//   straight into registers (64 tokens 198 us, 128 tokens 244 us).
// - N <= 128, row-major: logprob_stream_kernel. The same chunks with W through
//   LDS in whole cache lines; bound by HBM reading 128-byte pieces 8 KB apart
//   (64 tokens 279 -> 241 us, 128 tokens 339 -> 304 us; one 8-wave workgroup
//   per compute unit instead of two of 4 waves: 285 us at 64 tokens).
// - 128 < N < 512 over a small vocabulary: the two above, a block of 128 tokens a
//   workgroup (logprob_in_squares).
// - 128 < N < 512 otherwise: logprob_rounds_kernel. 256-token tiles, 384 vocabulary rows
//   high while they fill the 256 compute units, then lower ones for what is
//   left, so that the last round is short (row-major 129 tokens 464 -> 287 us,
//   256 526 -> 329, 257 658 -> 470, 400 814 -> 554, 511 870 -> 575; packed 129
//   tokens 367 -> 276, 256 402 -> 337, 257 519 -> 486, 511 715 -> 603 us; the
//   alternative being 128 x 128 tiles that load W again for every 128 tokens).
//   Blocks of 192 tokens where that holds the batch (257 tokens, row-major: 544
//   us in blocks of 256, 470 us in blocks of 192).
// - N >= 512: logprob_tile_kernel, 384 x 256 tiles with h staged. When the last
//   round of tiles would leave over half of the 256 compute units idle, its
//   tiles are cut along the tokens, 128 or 64 each, so that the round is short
//   too (its partial results stay where they are, one per token and chunk): 1,000
//   tokens 1,094 -> 1,073 us (48 tiles of 256 tokens became 192 of 64), 512
//   tokens 618 -> 597, 2,048 tokens 2,066 -> 2,042 us. Cutting them along D or
//   the vocabulary costs partial logits or partials.
//
// logprob_partial_kernel: each wave computes the logits of its 32 vocabulary
// rows for the batch's tokens on the matrix cores (4 or 2 tiles of
// mfma_f32_32x32x16_bf16: A = W rows, B = h^T). The loop walks D in steps of 64
// dims. W comes straight from memory, three steps ahead. The h slice (tokens x
// 64 dims) is requested two steps ahead, staged once per step into LDS
// (double-buffered, rows padded to 144 B: conflict-free) and read by all four
// waves. The 64 dims of a step are split over the four products as lanes 0-31
// dims 8u + 0..7 and lanes 32-63 dims 32 + 8u + 0..7 (any split of the
// contraction is valid as long as A and B use the same one). The wave reduces
// its logits to a (max, sum of exp) pair per token in base 2, the four waves
// merge through LDS, and the workgroup writes one partial per token; the
// workgroup whose chunk holds token n's target stores that logit.
//
// Combine kernel: one workgroup per token merges its partials:
// M = max_c m_c, L = sum_c l_c 2^(m_c - M), lse = (M + log2 L) ln 2.
//
// Packed LM head: W [V][D] row-major makes every wave read 32 rows 128 bytes
// at a time, 8 KB apart. The packed copy stores the matrix in the order the
// products consume it, [D/64][tiles][4][64 lanes][8] (32-row tiles, V rounded
// up to whole 384-row chunks): each load instruction reads 1 KB contiguous,
// a wave's step is 4 KB contiguous, and the waves working on one 64-dim step
// at the same time read one narrow window of memory rather than thousands of
// separate runs. Same products in the same order: the results are bitwise
// those of the row-major matrix.
#include "ra_device.h"
#include "ra_internal.h"

namespace ra {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kLpWaves = 4;
constexpr int kLpThreads = kLpWaves * kWave;
constexpr int kVocabChunk = 32 * kLpWaves;    // vocabulary rows per workgroup
constexpr int kMaxTiles = 4;                  // 32-token tiles per workgroup (largest variant)
constexpr int kDimStep = 64;                  // dims per loop step (4 products)
constexpr int kXcds = 8;                      // XCDs of an MI355X
constexpr int kHPitch = kDimStep + 8;         // LDS row pitch of the h slice (elements)
constexpr int kRoundsMinN = 128;              // larger batches below kTileMinN: tiles of two heights
constexpr int kTileCus = 256;                 // compute units of an MI355X, one tile each
constexpr int kTileMinN = 512;                // batches from this size use the 384 x 256 tiles
constexpr int64_t kMemorySideCache = 256 << 20;   // bytes
constexpr int kPackRows = 384;                // the packed copy covers V rounded up to this
// s_waitcnt immediates: vmcnt(0), export and LDS counters not waited on
constexpr int kWaitVm0 = 0x0F70;

struct LogprobArgs {
  const uint16_t *h;
  const uint16_t *hp;   // N >= kTileMinN: h in the tiled kernel's LDS stage order (workspace)
  const uint16_t *W;
  const int32_t *targets;
  float *ws_m;    // [N][chunks] running max, base-2 units
  float *ws_l;    // [N][chunks] sum of 2^(y - max)
  float *tgt;     // [N] logit of the target (natural units)
  int32_t N, V, D, chunks, token_blocks;
  int32_t tall;       // chunks of 384 rows in whole 256-token (or largest) tiles before the last round
  float scale;        // logits = scale * <h, W_v>
  float scale_log2;   // scale * log2(e)
};

__device__ __forceinline__ f32x16 mfma32x32x16(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// Max / sum over lanes l and l ^ 32 (v_permlane32_swap gives each lane both).
__device__ __forceinline__ float pair_max(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false,
                                                  false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float pair_sum(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false,
                                                  false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// (max, sum of 2^(y - max)) of token t's logits over the 32 vocabulary rows
// from v0 (lane l holds rows v0 + 8 (r / 4) + 4 half + r % 4, r = 0..15, of the
// token of column l % 32), and the target's logit if it is among them.
__device__ __forceinline__ void tile_max_sum(const LogprobArgs &a, const f32x16 &acc, int v0, int t,
                                             int half, float *max_out, float *sum_out) {
  const int target = t < a.N ? a.targets[t] : -1;
  float y[16];
  float m = -INFINITY;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int v = v0 + 8 * (r >> 2) + 4 * half + (r & 3);
    y[r] = v < a.V ? acc[r] * a.scale_log2 : -INFINITY;
    m = fmaxf(m, y[r]);
    if (v == target) a.tgt[t] = acc[r] * a.scale;
  }
  m = pair_max(m);
  const float m_use = m == -INFINITY ? 0.f : m;
  float sum = 0.f;
#pragma unroll
  for (int r = 0; r < 16; ++r) sum += fast_exp2(y[r] - m_use);
  *max_out = m;
  *sum_out = pair_sum(sum);
}

// Merges four waves' (max, sum) of column c into token t's partial of a chunk.
template <int kColumns>
__device__ __forceinline__ void merge_waves(const LogprobArgs &a, const float (*s_m)[kColumns],
                                            const float (*s_l)[kColumns], int c, int t, int chunk) {
  float M = s_m[0][c];
#pragma unroll
  for (int w = 1; w < kLpWaves; ++w) M = fmaxf(M, s_m[w][c]);
  const float M_use = M == -INFINITY ? 0.f : M;
  float L = 0.f;
#pragma unroll
  for (int w = 0; w < kLpWaves; ++w) L += s_l[w][c] * fast_exp2(s_m[w][c] - M_use);
  const size_t part = (size_t)t * a.chunks + chunk;
  a.ws_m[part] = M;
  a.ws_l[part] = L;
}

// kTiles 32-token tiles per workgroup: 2 for small batches (N <= 64), else 4.
template <int kTiles>
__global__ __launch_bounds__(kLpThreads, 2) void logprob_partial_kernel(LogprobArgs a) {
  constexpr int kTokenBlock = 32 * kTiles;
  // XCD-aware placement: workgroup ids are dealt to the XCDs round-robin, so
  // ids id, id + 8, id + 16, ... share an XCD; those consecutive "slots" get
  // the token blocks of one vocabulary chunk.
  const int id = blockIdx.x;
  const int xcd = id % kXcds, slot = id / kXcds;
  const int chunk = (slot / a.token_blocks) * kXcds + xcd;
  const int tblock = slot - (slot / a.token_blocks) * a.token_blocks;
  if (chunk >= a.chunks) return;

  const int lane = threadIdx.x & (kWave - 1);
  const int wave = threadIdx.x / kWave;
  const int col = lane & 31, half = lane >> 5;
  const int v0 = chunk * kVocabChunk + wave * 32;       // first vocabulary row of this wave
  const int t0 = tblock * kTokenBlock;                  // first token of the block

  // this lane's units of the packed copy (rows past V are stored as zeros and
  // masked after the products)
  const uint16_t *wp = a.W + (size_t)(v0 / 32) * 4 * kWave * 8 + 8 * lane;
  // h staging: thread i copies 16-byte chunks i + 256 j (j = 0..3) of the
  // block's 128 x 64 slice (token = chunk / 8, 8 dims per chunk); tokens past
  // N are clamped (their columns are never written back).
  constexpr int kHChunks = kTokenBlock * kDimStep / 8 / kLpThreads;   // 2 or 4
  __shared__ __attribute__((aligned(16))) uint16_t s_h[2][kTokenBlock * kHPitch];
  const uint16_t *hsrc[kHChunks];
  int hdst[kHChunks];
#pragma unroll
  for (int i = 0; i < kHChunks; ++i) {
    const int c = threadIdx.x + kLpThreads * i, tok = c >> 3, d8 = (c & 7) * 8;
    hsrc[i] = a.h + (size_t)min(t0 + tok, a.N - 1) * a.D + d8;
    hdst[i] = tok * kHPitch + d8;
  }
  // Two register sets for h (requested two steps ahead) and four for W
  // (three steps ahead); the loop body is four steps so that every set keeps
  // a fixed role and no operand is copied.
  u32x4 hx[kHChunks], hy[kHChunks];
  auto h_load = [&](u32x4 *dst, int s) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < kHChunks; ++i) dst[i] = load_u32x4(hsrc[i] + s * kDimStep);
  };
  auto h_store = [&](int buf, const u32x4 *src) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < kHChunks; ++i) store_u32x4(&s_h[buf][hdst[i]], src[i]);
  };
  // With one token block no other workgroup reads this chunk of W, and a
  // load takes 1 KB contiguous (whole cache lines): marked nontemporal for the
  // batches of 64 tokens, whose reads are all the time there is.
  constexpr bool kStreamW = kTiles == 2;
  // 32-row tiles of the packed copy: a 64-dim step of all of them is one block
  const size_t ntiles = (size_t)(((int64_t)a.V + kPackRows - 1) / kPackRows) * (kPackRows / 32);
  bf16x8 w0[4], w1[4], w2[4], w3[4];
  auto w_load = [&](bf16x8 *dst, int s) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < 4; ++u)
    {
      const uint16_t *p = wp + ((size_t)s * ntiles * 4 + u) * 8 * kWave;
      dst[u] = kStreamW ? __builtin_bit_cast(bf16x8, load_stream_u32x4(p)) : load_bf16x8(p);
    }
  };
  const int nsteps = a.D / kDimStep;
  const int last = nsteps - 1;
  f32x16 acc[kTiles];
#pragma unroll
  for (int tt = 0; tt < kTiles; ++tt) acc[tt] = f32x16{};
  // Step s: request h(s + 2) into `hf` and W(s + 3) into `wf` (past the last
  // step the requests repeat it: branch-free, exact wait counts), run the
  // products of step s on `wu` and LDS buffer s & 1, then store h(s + 1)
  // (register set `hs`) into the other buffer.
  auto step = [&](int s, const bf16x8 *wu, bf16x8 *wf, u32x4 *hf, const u32x4 *hs)
      __attribute__((always_inline)) {
    h_load(hf, min(s + 2, last));
    w_load(wf, min(s + 3, last));
    const uint16_t *hb = &s_h[s & 1][col * kHPitch + 32 * half];
#pragma unroll
    for (int tt = 0; tt < kTiles; ++tt) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const bf16x8 b = __builtin_bit_cast(
            bf16x8, *reinterpret_cast<const u32x4 *>(hb + 32 * tt * kHPitch + 8 * u));
        acc[tt] = mfma32x32x16(wu[u], b, acc[tt]);
      }
    }
    h_store((s + 1) & 1, hs);
    __syncthreads();
  };

  h_load(hx, 0);
  h_load(hy, min(1, last));
  w_load(w0, 0);
  w_load(w1, min(1, last));
  w_load(w2, min(2, last));
  h_store(0, hx);
  __syncthreads();
  // step s uses W set s % 4 and h register set (s + 1) % 2 for the store
  int s = 0;
  for (; s + 4 <= nsteps; s += 4) {
    step(s, w0, w3, hx, hy);
    step(s + 1, w1, w0, hy, hx);
    step(s + 2, w2, w1, hx, hy);
    step(s + 3, w3, w2, hy, hx);
  }
  if (s < nsteps) step(s, w0, w3, hx, hy);
  if (s + 1 < nsteps) step(s + 1, w1, w0, hy, hx);
  if (s + 2 < nsteps) step(s + 2, w2, w1, hx, hy);

  // Lane l holds, for token column t0 + 32 tt + col, the logits of vocabulary
  // rows v0 + 8 (r / 4) + 4 half + r % 4, r = 0..15.
  __shared__ float s_m[kLpWaves][kTokenBlock];
  __shared__ float s_l[kLpWaves][kTokenBlock];
#pragma unroll
  for (int tt = 0; tt < kTiles; ++tt) {
    float m, sum;
    tile_max_sum(a, acc[tt], v0, t0 + 32 * tt + col, half, &m, &sum);
    if (half == 0) {
      s_m[wave][32 * tt + col] = m;
      s_l[wave][32 * tt + col] = sum;
    }
  }
  __syncthreads();

  // Merge the four waves: one thread per token of the block.
  const int c = threadIdx.x;
  if (c < kTokenBlock && t0 + c < a.N) merge_waves(a, s_m, s_l, c, t0 + c, chunk);
}

// ---- large batches: LDS-tiled products, 384 vocabulary rows x 256 tokens ----
//
// At N >= kTileMinN one workgroup of 8 waves (one per compute unit) owns a
// 384 x 256 tile of logits (vocabulary rows x tokens). Each compute unit then
// loads 40 KB of W and h per 384 x 256 x 32 multiply-adds, about 19 % fewer
// bytes per product than a 256 x 256 tile and less than half of what the 128 x 128
// tiles above load; those are bound by how fast the L2 delivers operands to
// the compute units, not by the matrix cores. The loop walks D in steps of 32
// dims through a ring of 3 LDS stages (24 KB of W and 16 KB of h each),
// refilled two steps ahead by direct global-to-LDS loads
// (global_load_lds_dwordx4, no register staging); the five refill loads of a
// wave and step are spread between its products. Wave w computes rows
// 96 (w % 4) .. + 95 (three 32-row tiles) against tokens 128 (w / 4) .. + 127
// (four 32-token tiles): 24 products per step from 14 LDS operand reads, 192
// accumulator registers.
//
// Stage layout: row r of a region holds its 32 dims as four 16-byte chunks,
// logical chunk c at slot c ^ ((r / 4) % 4), so that 16 lanes reading 16 rows
// at one logical chunk hit 16 distinct bank groups. A load instruction fills
// 16 rows: lane l fetches row 16 j + l / 4, the logical chunk stored at slot
// l % 4.
// From the packed copy W keeps that copy's order instead: a 32-row tile is chunk 0 of its
// rows, then chunk 1, ...; a load instruction takes 512 contiguous bytes twice, where
// the row order took 16 bytes from each of 64 places (2,048 tokens 1,992 -> 1,936 us, 512
// tokens 594 -> 541 us, 257 tokens over 20,000 rows 81 -> 70 us).
// The 32 dims of a step split over the two products as lanes 0-31 dims
// 8 u + 0..7 and lanes 32-63 dims 16 + 8 u + 0..7 (logical chunk 2 half + u).
constexpr int kTileRows = 256;        // tokens per workgroup
constexpr int kTileRowsA = 384;       // vocabulary rows per workgroup
constexpr int kTileWaves = 8;
constexpr int kTileThreads = kTileWaves * kWave;
constexpr int kTileDims = 32;         // dims per step
constexpr int kTileStages = 3;
constexpr int kTileElems = kTileRows * kTileDims;     // token region of a stage (16 KB)
constexpr int kTileElemsA = kTileRowsA * kTileDims;   // vocabulary region (24 KB)
// Refill load d of a step goes after this one of the step's products.
template <int kLoads, int kProducts>
__device__ constexpr int load_after(int d) {
  if (kLoads == 5 && kProducts == 24) return d == 4 ? 22 : 3 + 5 * d;
  return (2 * d + 1) * kProducts / (2 * kLoads);
}

// Direct global-to-LDS load of 16 bytes per lane: lane l's bytes land at LDS
// address `lds` + 16 l (lds wave-uniform). Written out rather than through the
// compiler builtin, which makes the compiler wait for every such load before
// any LDS read (it cannot tell the ring's stages apart); the kernel counts
// its own loads. M0 is the LDS base register; named as clobbered instead of
// saved and restored around every load: 2,030 -> 2,026 us at 2,048 tokens of
// the Qwen3-8B head.
__device__ __forceinline__ uint32_t lds_address(const uint16_t *p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void *)p;
}
__device__ __forceinline__ void load_lds16(const uint16_t *g, uint32_t lds) {
  asm volatile(
      "s_mov_b32 m0, %0\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %1, off"
      :
      : "s"(lds), "v"(g)
      : "memory", "m0");
}
// The same, marked nontemporal: for data read once, a whole line at a time.
__device__ __forceinline__ void load_lds16_stream(const uint16_t *g, uint32_t lds) {
  asm volatile(
      "s_mov_b32 m0, %0\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %1, off nt"
      :
      : "s"(lds), "v"(g)
      : "memory", "m0");
}

// One tile: RT 32-row tiles per wave (128 RT vocabulary rows from v0) x TT
// 32-token tiles per wave (64 TT tokens: part `sub` of token block tblock),
// partial results into column `part`. kStagedH: h from
// its staged copy (the workspace holds one from N = kTileMinN on), otherwise
// from its rows, 64 bytes at a time like a row-major W.
struct TileLds {
  __attribute__((aligned(1024))) uint16_t a[kTileStages][kTileElemsA];
  __attribute__((aligned(1024))) uint16_t b[kTileStages][kTileElems];
  float m[4][kTileRows];
  float l[4][kTileRows];
};
template <bool kPacked, bool kStagedH, int RT, int TT>
__device__ __forceinline__ void logprob_tile(const LogprobArgs &a, int v0, int tblock, int sub,
                                             int part, TileLds &lds) {
  auto &sA = lds.a;
  auto &sB = lds.b;
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  constexpr int kTokens = 64 * TT;
  const int t0 = kStagedH ? tblock * kTileRows + sub * kTokens : tblock * kTokens;
  // load instructions (16 rows each) of a wave and step; of a 64-token tile's
  // four h instructions each is issued by two waves
  constexpr int kLoadsA = RT, kLoadsB = (TT + 1) / 2;

  // ---- loads: instructions kLoadsA * wave + k of the W region, kLoadsB *
  // wave + k of the h region ----
  const uint16_t *ga[kLoadsA], *gb[kLoadsB];
  // rows past the matrix (packed: past its copy, a multiple of 384 rows) read its last one
  const int vlast = kPacked ? (a.V + kPackRows - 1) / kPackRows * kPackRows - 1 : a.V - 1;
#pragma unroll
  for (int k = 0; k < kLoadsA; ++k) {
    const int j = kLoadsA * wave + k;
    if constexpr (kPacked) {
      // half a 32-row tile, chunks 2 (j % 2) and + 1 of every row: 16-byte units
      // ((s / 2 * tiles + tile) * 4 + lc) * 64 + 32 (s % 2) + row, 512 contiguous
      // bytes a chunk (the part that depends on the step s is added per step)
      const int tile = min(v0 / 32 + j / 2, vlast / 32), lc = 2 * (j & 1) + lane / 32;
      ga[k] = a.W + ((size_t)tile * 4 + lc) * kWave * 8 + (lane % 32) * 8;
    } else {
      const int r = 16 * j + lane / 4, lc = (lane % 4) ^ ((r >> 2) & 3);
      ga[k] = a.W + (size_t)min(v0 + r, vlast) * a.D + 8 * lc;
    }
  }
  const int nsteps = a.D / kTileDims;
  auto h_instr = [&](int k) __attribute__((always_inline)) {
    return TT == 1 ? wave % 4 : kLoadsB * wave + k;
  };
  // a staged copy of h holds each (token block, step) as the 16 KB image of
  // its LDS region: load instruction j reads 1 KB contiguous
#pragma unroll
  for (int k = 0; k < kLoadsB; ++k) {
    const int j = h_instr(k), r = 16 * j + lane / 4;
    const int lc = (lane % 4) ^ ((r >> 2) & 3);
    gb[k] = kStagedH ? a.hp + (size_t)tblock * nsteps * kTileElems + (size_t)(4 * TT * sub + j) * 512 +
                           lane * 8
                     : a.h + (size_t)min(t0 + min(r, kTokens - 1), a.N - 1) * a.D + 8 * lc;
  }
  const int last = nsteps - 1;
  const uint32_t blkA = (uint32_t)(kLoadsA * wave) * 1024u;
  // offsets (elements) of step s in W and h; steps past the last repeat it
  // (branch-free, so that every step issues the same number of loads)
  // elements per 64-dim step of the packed copy (all of its 32-row tiles)
  const size_t pstride =
      (size_t)(((int64_t)a.V + kPackRows - 1) / kPackRows) * (kPackRows / 32) * 4 * kWave * 8;
  auto w_off = [&](int s) __attribute__((always_inline)) {
    return kPacked ? (size_t)(s >> 1) * pstride + (s & 1) * 32 * 8 : (size_t)s * kTileDims;
  };
  auto load = [&](int st, int s, int d) __attribute__((always_inline)) {
    if (d < kLoadsA)
      load_lds16(ga[d] + w_off(s), lds_address(sA[st]) + blkA + 1024u * d);
    else
      load_lds16(gb[d - kLoadsA] + (size_t)s * (kStagedH ? kTileElems : kTileDims),
                 lds_address(sB[st]) + 1024u * h_instr(d - kLoadsA));
  };
  constexpr int kLoadsPerStep = kLoadsA + kLoadsB;
  constexpr int kProducts = 2 * RT * TT;
  // s_waitcnt vmcnt(kLoadsPerStep), export and LDS counters not waited on: one
  // later step's loads may stay in flight
  constexpr int kWaitStep = 0x0F70 | kLoadsPerStep;

  const int col = lane & 31, half = lane >> 5;
  const int wv = wave & 3, wt = wave >> 2;
  const int swz = (col >> 2) & 3;   // slot swizzle of every operand row (rows differ from col by multiples of 32)
  const int rowA = 32 * RT * wv * kTileDims + (kPacked ? 8 * col : kTileDims * col);
  const int rowB = (32 * TT * wt + col) * kTileDims;
  f32x16 acc[RT][TT];
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int j = 0; j < TT; ++j) acc[i][j] = f32x16{};
  auto lds16 = [](const uint16_t *p) __attribute__((always_inline)) {
    return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(p));
  };
  // Step s on stage st: wait until my loads for it have landed (the next
  // step's may still be in flight), barrier (everyone's have, and everyone is
  // done reading the stage used last step), then the products, with the
  // loads of step s + 2 into that freed stage spread between them.
  auto step = [&](int st, int s) __attribute__((always_inline)) {
    __builtin_amdgcn_s_waitcnt(kWaitStep);
    __builtin_amdgcn_s_barrier();
    const uint16_t *A = sA[st], *B = sB[st];
    const int rs = min(s + kTileStages - 1, last), rst = (st + kTileStages - 1) % kTileStages;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int c = 8 * ((2 * half + u) ^ swz);
      bf16x8 av[RT], bv[TT];
#pragma unroll
      for (int i = 0; i < RT; ++i)
        av[i] = lds16(A + rowA + (kPacked ? 32 * 8 * (2 * half + u) : c) + 32 * kTileDims * i);
#pragma unroll
      for (int j = 0; j < TT; ++j) bv[j] = lds16(B + rowB + c + 32 * kTileDims * j);
#pragma unroll
      for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < TT; ++j) {
          acc[i][j] = mfma32x32x16(av[i], bv[j], acc[i][j]);
          const int p = TT * (RT * u + i) + j;   // product index in the step
#pragma unroll
          for (int d = 0; d < kLoadsPerStep; ++d)
            if (p == load_after<kLoadsPerStep, kProducts>(d)) {
              __builtin_amdgcn_sched_barrier(0);
              load(rst, rs, d);
              __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
  };
#pragma unroll
  for (int k = 0; k < kTileStages - 1; ++k)
#pragma unroll
    for (int d = 0; d < kLoadsPerStep; ++d) load(k, min(k, last), d);
  for (int s = 0; s < nsteps; s += kTileStages) {
#pragma unroll
    for (int k = 0; k < kTileStages; ++k)
      if (s + k < nsteps) step(k, s + k);
  }
  // the last loads (repeats of the last step) must land before the
  // workgroup's LDS is released
  __builtin_amdgcn_s_waitcnt(kWaitVm0);

  // ---- logits -> (max, sum) per token over this wave's 32 RT rows ----
  // Lane l holds, for token t0 + 32 (TT wt + j) + col, the logits of rows
  // v0 + 32 (RT wv + i) + 8 (r / 4) + 4 half + r % 4, r = 0..15.
#pragma unroll
  for (int j = 0; j < TT; ++j) {
    const int tc = 32 * (TT * wt + j) + col, t = t0 + tc;
    const int target = t < a.N ? a.targets[t] : -1;
    float y[RT][16];
    float m = -INFINITY;
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int v = v0 + 32 * (RT * wv + i) + 8 * (r >> 2) + 4 * half + (r & 3);
        y[i][r] = v < a.V ? acc[i][j][r] * a.scale_log2 : -INFINITY;
        m = fmaxf(m, y[i][r]);
        if (v == target) a.tgt[t] = acc[i][j][r] * a.scale;
      }
    m = pair_max(m);
    const float m_use = m == -INFINITY ? 0.f : m;
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) sum += fast_exp2(y[i][r] - m_use);
    sum = pair_sum(sum);
    if (half == 0) {
      lds.m[wv][tc] = m;
      lds.l[wv][tc] = sum;
    }
  }
  __syncthreads();
  // merge the four row groups: one thread per token of the tile
  const int c = threadIdx.x;
  if (c < kTokens && t0 + c < a.N) {
    float M = lds.m[0][c];
#pragma unroll
    for (int w = 1; w < 4; ++w) M = fmaxf(M, lds.m[w][c]);
    const float M_use = M == -INFINITY ? 0.f : M;
    float L = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) L += lds.l[w][c] * fast_exp2(lds.m[w][c] - M_use);
    const size_t at = (size_t)(t0 + c) * a.chunks + part;
    a.ws_m[at] = M;
    a.ws_l[at] = L;
  }
}

// `tall` chunks in 256-token tiles, then the rest in tiles of 64 TT tokens.
template <bool kPacked, int TT>
__global__ __launch_bounds__(kTileThreads, 1) void logprob_tile_kernel(LogprobArgs a) {
  __shared__ TileLds lds;
  const int whole = a.tall * a.token_blocks;
  const bool split = TT != 4 && (int)blockIdx.x >= whole;   // (256-token tiles: none are cut)
  const int id = blockIdx.x - (split ? whole : 0), parts = split ? 4 / TT : 1;
  const int xcd = id % kXcds, slot = id / kXcds, per = a.token_blocks * parts;
  const int chunk = (split ? a.tall : 0) + (slot / per) * kXcds + xcd;
  const int s = slot - (slot / per) * per;
  if (chunk >= a.chunks) return;
  if (!split)
    logprob_tile<kPacked, true, 3, 4>(a, chunk * kTileRowsA, s, 0, chunk, lds);
  else if constexpr (TT != 4)
    logprob_tile<kPacked, true, 3, TT>(a, chunk * kTileRowsA, s / parts, s % parts, chunk, lds);
}

// Tiles of two heights: `tall` chunks of 384 rows, then chunks of 128 RT rows.
template <bool kPacked, int RT, int TT>
__global__ __launch_bounds__(kTileThreads, 1) void logprob_rounds_kernel(LogprobArgs a) {
  const int id = blockIdx.x;
  const int xcd = id % kXcds, slot = id / kXcds;
  const int chunk = (slot / a.token_blocks) * kXcds + xcd;
  const int tblock = slot - (slot / a.token_blocks) * a.token_blocks;
  if (chunk >= a.chunks) return;
  __shared__ TileLds lds;
  if (RT == 3 || chunk < a.tall)
    logprob_tile<kPacked, false, 3, TT>(a, chunk * kTileRowsA, tblock, 0, chunk, lds);
  else
    logprob_tile<kPacked, false, RT, TT>(
        a, a.tall * kTileRowsA + (chunk - a.tall) * 128 * RT, tblock, 0, chunk, lds);
}

// ---- small batches over a row-major W: one pass of W through LDS ----
//
// kWaves waves, each with 32 vocabulary rows and a block of 32 T tokens. The
// loop walks D in steps of 64 dims through a ring of kStages LDS stages, refilled
// kStages - 1 steps ahead by direct global-to-LDS loads of eight rows x 128
// bytes: whole cache lines, where operand loads straight into registers take
// each line 16 bytes at a time (a lane needs 16 bytes of its own row).
// Products, their order and the partial results are those of
// logprob_partial_kernel. kNt: W is marked nontemporal, for heads that the 256 MB
// memory-side cache cannot hold between calls (64 tokens at 151,936 x 4,096 264 -> 242
// us); one that fits stays there (at 32,000 x 4,096 58 us nontemporal, 43 us not).
//
// Stage layout: row r holds its 64 dims as eight 16-byte chunks, logical chunk c
// at slot c ^ ((r / 2) % 8), so that 16 lanes reading 16 rows at one logical
// chunk hit 16 distinct bank groups.
template <int T, int kWaves, int kStages, bool kNt>
__global__ __launch_bounds__(kWaves *kWave, 1) void logprob_stream_kernel(LogprobArgs a) {
  constexpr int kTokens = 32 * T, kRows = 32 * kWaves;
  constexpr int kLoadsW = 4, kLoadsH = kTokens / 8 / kWaves;   // per wave and step
  constexpr int kLoads = kLoadsW + kLoadsH;
  static_assert(kLoadsH * 8 * kWaves == kTokens && kLoads * (kStages - 2) < 16, "load counts");
  __shared__ __attribute__((aligned(1024))) uint16_t sW[kStages][kRows * kDimStep];
  __shared__ __attribute__((aligned(1024))) uint16_t sH[kStages][kTokens * kDimStep];
  __shared__ float s_m[kWaves][kTokens];
  __shared__ float s_l[kWaves][kTokens];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int col = lane & 31, half = lane >> 5;
  // the token blocks of one stretch of the vocabulary on one XCD, as in logprob_partial_kernel
  constexpr int kChunks = kWaves / kLpWaves;   // 128-row chunks of a workgroup
  const int id = blockIdx.x, xcd = id % kXcds, slot = id / kXcds;
  const int block = (slot / a.token_blocks) * kXcds + xcd;
  const int t0 = (slot - (slot / a.token_blocks) * a.token_blocks) * kTokens;
  if (block * kChunks >= a.chunks) return;
  const int v0 = (block * kWaves + wave) * 32;   // first vocabulary row of this wave

  const uint16_t *gw[kLoadsW], *gh[kLoadsH];
#pragma unroll
  for (int k = 0; k < kLoadsW; ++k) {
    const int r = 8 * k + lane / 8, lc = (lane % 8) ^ ((r >> 1) & 7);
    gw[k] = a.W + (size_t)min(v0 + r, a.V - 1) * a.D + 8 * lc;
  }
#pragma unroll
  for (int k = 0; k < kLoadsH; ++k) {
    const int r = 8 * (kLoadsH * wave + k) + lane / 8, lc = (lane % 8) ^ ((r >> 1) & 7);
    gh[k] = a.h + (size_t)min(t0 + r, a.N - 1) * a.D + 8 * lc;
  }
  const int nsteps = a.D / kDimStep, last = nsteps - 1;
  auto load = [&](int st, int s) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < kLoadsW; ++k)
      (kNt ? load_lds16_stream : load_lds16)(gw[k] + (size_t)s * kDimStep,
                                             lds_address(sW[st]) + (4 * wave + k) * 1024u);
#pragma unroll
    for (int k = 0; k < kLoadsH; ++k)
      load_lds16(gh[k] + (size_t)s * kDimStep, lds_address(sH[st]) + (kLoadsH * wave + k) * 1024u);
  };
  f32x16 acc[T];
#pragma unroll
  for (int tt = 0; tt < T; ++tt) acc[tt] = f32x16{};
  const int swz = (col >> 1) & 7;
  auto lds16 = [](const uint16_t *p) __attribute__((always_inline)) {
    return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(p));
  };
  // Step s on stage st: my loads for it have landed (those of kStages - 2 later
  // steps may be in flight), then everyone's have, and everyone is done with
  // the stage of the last step, which is refilled.
  auto step = [&](int st, int s) __attribute__((always_inline)) {
    __builtin_amdgcn_s_waitcnt(0x0F70 | (kLoads * (kStages - 2)));
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    load((st + kStages - 1) % kStages, min(s + kStages - 1, last));
    __builtin_amdgcn_sched_barrier(0);
    const uint16_t *A = sW[st] + (32 * wave + col) * kDimStep, *B = sH[st] + col * kDimStep;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int c = 8 * ((4 * half + u) ^ swz);
      const bf16x8 av = lds16(A + c);
#pragma unroll
      for (int tt = 0; tt < T; ++tt)
        acc[tt] = mfma32x32x16(av, lds16(B + c + 32 * kDimStep * tt), acc[tt]);
    }
  };
#pragma unroll
  for (int k = 0; k < kStages - 1; ++k) load(k, min(k, last));
  for (int s = 0; s < nsteps; s += kStages) {
#pragma unroll
    for (int k = 0; k < kStages; ++k)
      if (s + k < nsteps) step(k, s + k);
  }
  // the last loads (repeats of the last step) must land before the
  // workgroup's LDS is released
  __builtin_amdgcn_s_waitcnt(kWaitVm0);

#pragma unroll
  for (int tt = 0; tt < T; ++tt) {
    float m, sum;
    tile_max_sum(a, acc[tt], v0, t0 + 32 * tt + col, half, &m, &sum);
    if (half == 0) {
      s_m[wave][32 * tt + col] = m;
      s_l[wave][32 * tt + col] = sum;
    }
  }
  __syncthreads();
  // merge four waves (128 rows) into a partial: one thread per token and chunk
  for (int i = threadIdx.x; i < kTokens * kChunks; i += kWaves * kWave) {
    const int c = i % kTokens, g = i / kTokens, chunk = block * kChunks + g;
    if (t0 + c < a.N && chunk < a.chunks)
      merge_waves(a, &s_m[g * kLpWaves], &s_l[g * kLpWaves], c, t0 + c, chunk);
  }
}

// h staged for the tiled kernel: 16-byte unit u = ((tb * steps + s) * 256 + r) * 4
// + slot holds token 256 tb + r (zeros past N), dims 32 s + 8 (slot ^ ((r / 4) % 4))
// + 0..7 -- the LDS image of token block tb's step s.
__global__ __launch_bounds__(256) void logprob_stage_h_kernel(const uint16_t *__restrict__ h,
                                                              int32_t N, int32_t D, size_t units,
                                                              uint16_t *__restrict__ hp) {
  const size_t steps = (size_t)(D / kTileDims);
  for (size_t u = (size_t)blockIdx.x * blockDim.x + threadIdx.x; u < units;
       u += (size_t)gridDim.x * blockDim.x) {
    const int slot = (int)(u & 3);
    const size_t row = u >> 2;
    const int r = (int)(row % kTileRows);
    const size_t q = row / kTileRows, s = q % steps, tb = q / steps;
    const size_t t = tb * kTileRows + r;
    const int lc = slot ^ ((r >> 2) & 3);
    u32x4 v = {0u, 0u, 0u, 0u};
    if (t < (size_t)N) v = load_u32x4(h + t * D + kTileDims * s + 8 * lc);
    store_u32x4(hp + 8 * u, v);
  }
}

// Packed copy of W: 16-byte unit i = ((s * tiles + tile) * 4 + u) * 64 + lane
// holds W[32 tile + lane % 32][64 s + 32 (lane / 32) + 8 u + 0..7] (zeros for
// rows past V; tiles = the copy's rows / 32).
__global__ __launch_bounds__(256) void logprob_pack_kernel(const uint16_t *__restrict__ W,
                                                           int32_t V, int32_t D, size_t units,
                                                           uint16_t *__restrict__ Wp) {
  const size_t steps = (size_t)(D / kDimStep);
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < units;
       i += (size_t)gridDim.x * blockDim.x) {
    const int lane = (int)(i % kWave), u = (int)((i / kWave) % 4);
    const size_t ntiles = units / (4 * kWave * steps);
    const size_t tile = (i / (4 * kWave)) % ntiles, s = i / (4 * kWave * ntiles);
    const size_t row = 32 * tile + (lane & 31);
    const size_t dim = kDimStep * s + 32 * (lane >> 5) + 8 * u;
    u32x4 v = {0u, 0u, 0u, 0u};
    if (row < (size_t)V) v = load_u32x4(W + row * D + dim);
    store_u32x4(Wp + 8 * i, v);
  }
}

__global__ __launch_bounds__(kLpThreads) void logprob_combine_kernel(LogprobArgs a, float *logp,
                                                                   float *lse) {
  // One workgroup per token: thread i folds chunks i, i + 256, ... in order;
  // the lanes of a wave are combined by a fixed butterfly and the four waves
  // in wave order, so the result does not depend on timing.
  __shared__ float s_red[2][kLpWaves];
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int t = blockIdx.x;
  const float *m = a.ws_m + (size_t)t * a.chunks;
  const float *l = a.ws_l + (size_t)t * a.chunks;
  float M = -INFINITY;
  for (int c = threadIdx.x; c < a.chunks; c += kLpThreads) M = fmaxf(M, m[c]);
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) M = fmaxf(M, __shfl_xor(M, o));
  if (lane == 0) s_red[0][wave] = M;
  __syncthreads();
  M = fmaxf(fmaxf(s_red[0][0], s_red[0][1]), fmaxf(s_red[0][2], s_red[0][3]));
  float L = 0.f;
  for (int c = threadIdx.x; c < a.chunks; c += kLpThreads) L += l[c] * fast_exp2(m[c] - M);
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) L += __shfl_xor(L, o);
  if (lane == 0) s_red[1][wave] = L;
  __syncthreads();
  if (threadIdx.x == 0) {
    L = ((s_red[1][0] + s_red[1][1]) + s_red[1][2]) + s_red[1][3];
    const float ls = (M + __log2f(L)) * kLn2;
    const int target = a.targets[t];
    logp[t] = target >= 0 && target < a.V ? a.tgt[t] - ls : __builtin_nanf("");
    if (lse) lse[t] = ls;
  }
}

}  // namespace

namespace {
// Token blocks of 256 tokens and how the vocabulary is cut for them: `tall`
// chunks of 384 rows, then `rest` chunks of 128 `rt` rows.
struct Rounds {
  int32_t tall, rt, rest;
};
Rounds logprob_rounds(int32_t token_blocks, int32_t V) {
  const int64_t units = ((int64_t)V + 127) / 128;
  const int64_t per_round = kTileCus / token_blocks;   // chunks that run at the same time
  Rounds r;
  const int64_t full = units / 3 / per_round;          // rounds of 384-row chunks only
  r.tall = (int32_t)(full * per_round);
  const int64_t left = units - 3 * (int64_t)r.tall;
  r.rt = (int32_t)((left + per_round - 1) / per_round);
  if (r.rt < 1) r.rt = 1;
  if (r.rt > 3) r.rt = 3;
  r.rest = (int32_t)((left + r.rt - 1) / r.rt);
  return r;
}
// N >= kTileMinN: `whole` chunks (a multiple of 8) in 256-token tiles, the rest in
// tiles of 64 groups tokens when those still fit the compute units at once.
struct LastRound {
  int32_t whole;
  int groups;
};
LastRound logprob_last_round(int32_t token_blocks, int32_t chunks) {
  const int64_t tiles = (int64_t)chunks * token_blocks;
  LastRound r;
  r.whole = (int32_t)(tiles / kTileCus * kTileCus / token_blocks / kXcds * kXcds);
  const int64_t rest = (int64_t)(chunks - r.whole) * token_blocks;
  r.groups = rest == 0 || rest > kTileCus / 2 ? 4 : rest > kTileCus / 4 ? 2 : 1;
  return r;
}
int32_t token_blocks_of(int32_t N) { return (N + kTileRows - 1) / kTileRows; }
// Batches of few tiles: 128 x 128, when all of them run at once, one a compute unit, and
// the blocks of 192 or 256 tokens are fuller than kSquareTokens on average. Then a step's
// chain is what a tile takes, and the smaller tile's is shorter (4,096 x 4,096, row-major:
// 256 tokens 55 us in tiles of 256 tokens, 43 us in squares, 384 tokens 54 and 43 us; packed
// 52 and 46 us, 46 and 46 us); emptier blocks are no slower than squares (257 tokens 45 and
// 44 us, packed 45 and 47 us).
constexpr int kSquareTokens = 140;
bool logprob_in_squares(int32_t N, int32_t V) {
  if (N <= kRoundsMinN) return true;
  return N < kTileMinN && N > kSquareTokens * token_blocks_of(N) &&
         ((int64_t)V + 127) / 128 * ((N + 127) / 128) <= kTileCus;
}
bool logprob_in_rounds(int32_t N, int32_t V) { return N < kTileMinN && !logprob_in_squares(N, V); }
// 64-token groups of a token block (3 or 4)
int rounds_groups(int32_t N) {
  const int blocks = token_blocks_of(N);
  return (N + 64 * blocks - 1) / (64 * blocks) <= 3 ? 3 : 4;
}
}  // namespace

int32_t logprob_chunks(int32_t N, int32_t V) {
  if (logprob_in_rounds(N, V)) {
    const Rounds r = logprob_rounds(token_blocks_of(N), V);
    return r.tall + r.rest;
  }
  const int rows = N >= kTileMinN ? kTileRowsA : kVocabChunk;
  return (int32_t)(((int64_t)V + rows - 1) / rows);
}

// The packed copy covers every row a workgroup reads: V rounded up to whole
// 384-row chunks (so to whole 128-row chunks too).
size_t logprob_packed_bytes(int32_t V, int32_t D) {
  return (size_t)(((int64_t)V + kPackRows - 1) / kPackRows) * kPackRows * D * sizeof(uint16_t);
}

hipError_t launch_logprob_pack(const uint16_t *W, int32_t V, int32_t D, uint16_t *Wp,
                               hipStream_t stream) {
  const size_t units = logprob_packed_bytes(V, D) / 16;
  const size_t want = (units + 255) / 256, blocks = want < 65536 ? want : 65536;
  hipLaunchKernelGGL(logprob_pack_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, W, V, D,
                     units, Wp);
  return hipGetLastError();
}

namespace {
// per-(token, chunk) partials and the target logits (below kTileMinN at the
// 128-row chunks of the smallest batches, the most any batch there has)
size_t logprob_partial_bytes(int32_t N, int32_t V) {
  const int rows = N >= kTileMinN ? kTileRowsA : kVocabChunk;
  const size_t chunks = ((size_t)V + rows - 1) / rows;
  return ((size_t)N * chunks * 2 + (size_t)N) * sizeof(float);
}
}  // namespace

// The partials, then (from N = kTileMinN) the staged copy of h at the next
// 256-byte boundary: N rounded up to whole 256-token blocks x D bf16.
size_t logprob_workspace_bytes(int32_t N, int32_t V, int32_t D) {
  const size_t partials = (logprob_partial_bytes(N, V) + 255) / 256 * 256;
  if (N < kTileMinN) return logprob_partial_bytes(N, V);
  return partials + (size_t)((N + kTileRows - 1) / kTileRows) * kTileRows * D * sizeof(uint16_t);
}

namespace {
int logprob_tiles(int32_t N) { return N <= 64 ? 2 : kMaxTiles; }
// tokens per workgroup
int logprob_token_block(int32_t N, int32_t V) {
  if (logprob_in_rounds(N, V)) return 64 * rounds_groups(N);
  return N >= kTileMinN ? kTileRows : 32 * logprob_tiles(N);
}
}  // namespace

int64_t logprob_grid(int32_t N, int32_t V) {
  const int64_t chunks_pad = (logprob_chunks(N, V) + kXcds - 1) / kXcds * kXcds;
  const int block = logprob_token_block(N, V);
  return chunks_pad * ((N + block - 1) / block);
}

hipError_t launch_logprob(const uint16_t *h, const uint16_t *W, const int32_t *targets, int32_t N,
                          int32_t V, int32_t D, float scale, float *logp, float *lse,
                          void *workspace, bool packed, hipStream_t stream) {
  LogprobArgs a;
  a.h = h;
  a.hp = nullptr;
  a.W = W;
  a.targets = targets;
  a.N = N;
  a.V = V;
  a.D = D;
  a.chunks = logprob_chunks(N, V);
  const int tiles = logprob_tiles(N);
  const int block = logprob_token_block(N, V);
  a.token_blocks = (N + block - 1) / block;
  a.ws_m = static_cast<float *>(workspace);
  a.ws_l = a.ws_m + (size_t)N * a.chunks;
  a.tgt = a.ws_l + (size_t)N * a.chunks;
  a.scale = scale;
  a.scale_log2 = scale * kLog2e;
  const dim3 grid((unsigned)logprob_grid(N, V));
  if (N >= kTileMinN) {
    uint16_t *hp = reinterpret_cast<uint16_t *>(static_cast<char *>(workspace) +
                                                (logprob_partial_bytes(N, V) + 255) / 256 * 256);
    a.hp = hp;
    const size_t units = (size_t)a.token_blocks * kTileRows * D / 8;
    const size_t want = (units + 255) / 256, blocks = want < 65536 ? want : 65536;
    hipLaunchKernelGGL(logprob_stage_h_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, h, N,
                       D, units, hp);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  a.tall = 0;
  if (logprob_in_rounds(N, V)) {
    const Rounds r = logprob_rounds(a.token_blocks, V);
    a.tall = r.tall;
    const int variant = (packed ? 6 : 0) + (rounds_groups(N) == 4 ? 3 : 0) + r.rt - 1;
    switch (variant) {
#define RA_ROUNDS(X, P, RT, TT)                                                                   \
  case X:                                                                                         \
    hipLaunchKernelGGL((logprob_rounds_kernel<P, RT, TT>), grid, dim3(kTileThreads), 0, stream, a); \
    break;
      RA_ROUNDS(0, false, 1, 3)
      RA_ROUNDS(1, false, 2, 3)
      RA_ROUNDS(2, false, 3, 3)
      RA_ROUNDS(3, false, 1, 4)
      RA_ROUNDS(4, false, 2, 4)
      RA_ROUNDS(5, false, 3, 4)
      RA_ROUNDS(6, true, 1, 3)
      RA_ROUNDS(7, true, 2, 3)
      RA_ROUNDS(8, true, 3, 3)
      RA_ROUNDS(9, true, 1, 4)
      RA_ROUNDS(10, true, 2, 4)
      RA_ROUNDS(11, true, 3, 4)
#undef RA_ROUNDS
    }
  } else if (N >= kTileMinN) {
    const LastRound r = logprob_last_round(a.token_blocks, a.chunks);
    a.tall = r.whole;
    const int64_t rest = (a.chunks - r.whole + kXcds - 1) / kXcds * kXcds;
    const dim3 tiles = r.groups == 4 ? grid
                                     : dim3((unsigned)(((int64_t)r.whole + rest * (4 / r.groups)) *
                                                       a.token_blocks));
    switch ((packed ? 3 : 0) + (r.groups == 4 ? 2 : r.groups - 1)) {
#define RA_TILES(X, P, TT)                                                                       \
  case X:                                                                                        \
    hipLaunchKernelGGL((logprob_tile_kernel<P, TT>), tiles, dim3(kTileThreads), 0, stream, a); \
    break;
      RA_TILES(0, false, 1)
      RA_TILES(1, false, 2)
      RA_TILES(2, false, 4)
      RA_TILES(3, true, 1)
      RA_TILES(4, true, 2)
      RA_TILES(5, true, 4)
#undef RA_TILES
    }
  }
  else if (packed && tiles == 2)
    hipLaunchKernelGGL((logprob_partial_kernel<2>), grid, dim3(kLpThreads), 0, stream, a);
  else if (packed)
    hipLaunchKernelGGL((logprob_partial_kernel<kMaxTiles>), grid, dim3(kLpThreads), 0, stream, a);
  else {
    // Row-major. 64 tokens: 72 KB of LDS, two workgroups per compute unit. More: workgroups
    // of 4 waves while those of 8 would leave compute units idle (at most 256 chunks:
    // 128 tokens at 32,000 x 4,096 72 us with 8 waves, 50 us with 4).
    const bool nt = (int64_t)V * D * (int64_t)sizeof(uint16_t) > kMemorySideCache;
    const int waves = tiles == 2 || a.chunks <= kTileCus ? 4 : 8;
    const dim3 g(waves == 4 ? grid.x : (unsigned)((a.chunks + 1) / 2 + kXcds - 1) / kXcds * kXcds);
    const dim3 b(waves * kWave);
    const int variant = (tiles == 2 ? 0 : waves) | (nt ? 1 : 0);
    switch (variant) {
#define RA_STREAM(X, T, W, NT)                                                        \
  case X:                                                                             \
    hipLaunchKernelGGL((logprob_stream_kernel<T, W, 3, NT>), g, b, 0, stream, a);     \
    break;
      RA_STREAM(0, 2, 4, false)
      RA_STREAM(1, 2, 4, true)
      RA_STREAM(4, kMaxTiles, 4, false)
      RA_STREAM(5, kMaxTiles, 4, true)
      RA_STREAM(8, kMaxTiles, 8, false)
      RA_STREAM(9, kMaxTiles, 8, true)
#undef RA_STREAM
    }
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(logprob_combine_kernel, dim3((unsigned)N), dim3(kLpThreads), 0, stream, a,
                     logp, lse);
  return hipGetLastError();
}

}  // namespace ra
