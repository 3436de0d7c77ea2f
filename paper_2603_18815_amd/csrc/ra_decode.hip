// Decode attention over paged KV caches: split-K over pages, then combine.
// The split and the combine are described with decode_split in the header.
#include <stdlib.h>

#include "ra_decode_split.h"
#include "ra_internal.h"

namespace ra {
namespace {

using namespace dsplit;

constexpr int kSplitWaves = 4;

// KV head fastest: the Hkv workgroups of one (item, split) are dispatched
// together, so the Hkv adjacent 4 KiB blocks of every page they read are
// requested close in time (DRAM row locality).
// kDirect: every row is one split, whose result goes to out and lse.
template <int NT, bool kFp8, bool kDirect>
__global__ __launch_bounds__(kSplitWaves * kWave, 2) void decode_split_kernel(DecodeArgs a,
                                                                             float *out,
                                                                             float *lse) {
  __shared__ DecodeLds<NT, kSplitWaves> lds;
  decode_split<NT, false, kSplitWaves, kFp8, kDirect>(a, blockIdx.x, blockIdx.y, blockIdx.z, lds,
                                                      out, lse);
}

// Shared-prefix decode in one launch. Planes z < prefix_planes hold the
// prefix items, item i = z * gridDim.y + y, with the chunks of one (group,
// prefix split) adjacent so that the workgroups reading the same prefix pages
// run close together (the later ones mostly hit the cache); the planes after
// hold the row items as in plain decode. One launch lets the few prefix items
// run beside the many row items instead of before them, in a pass of their own
// that leaves most of the machine idle.
template <int NT, bool kFp8>
__global__ __launch_bounds__(kSplitWaves * kWave, 2) void decode_shared_kernel(
    DecodeArgs a, int32_t prefix_planes, int32_t chunks, int32_t prefix_items) {
  __shared__ DecodeLds<NT, kSplitWaves> lds;
  const int z = blockIdx.z;
  if (z < prefix_planes) {
    const int i = z * gridDim.y + blockIdx.y;
    if (i >= prefix_items) return;
    const int sub = i % chunks, gs = i / chunks;
    const int split = gs % a.prefix_slots, grp = gs / a.prefix_slots;
    DecodeArgs p = a;
    p.zdiv = chunks;
    decode_split<NT, true, kSplitWaves, kFp8>(p, blockIdx.x, split, grp * chunks + sub, lds);
  } else {
    decode_split<NT, false, kSplitWaves, kFp8>(a, blockIdx.x, blockIdx.y, z - prefix_planes, lds);
  }
}

template <int NT>
void launch_shared(bool fp8, dim3 grid, const DecodeArgs &a, const SharedPrefixShape &sh,
                   hipStream_t stream) {
  const int32_t planes = (int32_t)sh.prefix_planes, items = (int32_t)sh.prefix_items;
  if (fp8)
    hipLaunchKernelGGL((decode_shared_kernel<NT, true>), grid, dim3(kSplitWaves * kWave), 0,
                       stream, a, planes, sh.chunks, items);
  else
    hipLaunchKernelGGL((decode_shared_kernel<NT, false>), grid, dim3(kSplitWaves * kWave), 0,
                       stream, a, planes, sh.chunks, items);
}

template <int NT, bool kDirect>
void launch_split(bool fp8, dim3 grid, const DecodeArgs &a, float *out, float *lse,
                  hipStream_t stream) {
  if (fp8)
    hipLaunchKernelGGL((decode_split_kernel<NT, true, kDirect>), grid, dim3(kSplitWaves * kWave), 0,
                       stream, a, out, lse);
  else
    hipLaunchKernelGGL((decode_split_kernel<NT, false, kDirect>), grid, dim3(kSplitWaves * kWave), 0,
                       stream, a, out, lse);
}

// Split length forced by the environment (RA_SPLIT_TOKENS, for testing the
// split and combine paths), read once per process: a decimal number of keys
// in [128, 65536], rounded up to a multiple of 128; anything else (absent,
// not a number, out of range) leaves the planned length. 0 when unset.
int64_t split_override() {
  static const int64_t value = [] {
    const char *env = getenv("RA_SPLIT_TOKENS");
    if (!env || !*env) return (int64_t)0;
    char *end = nullptr;
    const long long v = strtoll(env, &end, 10);
    if (*end != '\0' || v < 128 || v > 65536) return (int64_t)0;
    return (int64_t)((v + 127) / 128 * 128);
  }();
  return value;
}

}  // namespace

// Calls with few (row, KV head) pairs (measured by graph replay, device time):
// - rows of at most kDirectKeys keys are one split, whose workgroup writes the
//   final result: no partials, no combine launch (4 rows of 32..256 keys 9.4 ->
//   6.6 us, 64 rows of 100..500 keys 23.0 -> 19.1 us). At 300 keys two splits and
//   a combine measure the same (7.4 against 7.5 us).
// - longer rows are split down to 128 keys while there are fewer than kSmallItems
//   items of the longest row's length: a split's four waves then take one page
//   pair each instead of four in a chain (1 row of 1,000 keys, 8 KV heads: 12.4
//   -> 7.6 us; 1 row of 4,096: 12.6 -> 8.8 us). Above that the shorter splits
//   only add partials (2 rows of 16,000: 27.3 us with 512-key splits, 30.4 with
//   256; 1 row of 65,000: 54 and 65 us). Splits are shortened below 512 keys only as
//   far as the longest row then has kSmallSlots slots (in 512-key splits it can have
//   more): its combine reads them in rounds (1 row of 30,000 keys, 1 KV head: 17.4 us
//   with 59 slots, 29.4 with 235; 1 row of 8,000, 2 KV heads: 10.2 with 32 slots, 11.1
//   with 63, 13.2 with 16). Nor are there to be more than
//   kSmallParts (head, slot) partials, which groups of 17 to 32 heads reach first
//   (8 rows of 4,000 keys, 32 heads over one KV head, 8,192 partials: 17.2 -> 14.4 us;
//   16 such rows 18.7 us in 512-key splits, 20.0 in 128-key ones, their shared-prefix
//   call 21.1 and 30.2; 64 rows of 600 keys, 10,240 partials: 18.1 -> 17.6 us).
constexpr int kDirectKeys = 512;
constexpr int kSmallItems = 256;
constexpr int kSmallSlots = 32;
constexpr int kSmallParts = 10240;

DecodePlan decode_plan(int32_t B, int32_t hkv, int32_t max_kv_len, int32_t group) {
  // Aim for about 8k (row, KV head, split) items on the longest-row bound:
  // enough workgroups to balance rows of different lengths over 256 CUs,
  // long enough splits that the partial results stay well under 1 % of the
  // KV bytes. Split lengths are powers of two in [512, 4096] keys (from 128 for
  // the few items above), multiples of 128 keys (4 waves x one page pair), and
  // depend only on the host-side sizes, never on page ids.
  int64_t work = (int64_t)B * hkv * (int64_t)(max_kv_len > 0 ? max_kv_len : 1);
  int64_t split = 512;
  while (split < 4096 && work / split > 8192) split *= 2;
  if (group > 0 && max_kv_len > kDirectKeys) {
    auto parts = [&](int64_t tokens) {
      return (int64_t)B * hkv * group * ((max_kv_len + tokens - 1) / tokens);
    };
    while (split > 128 && work / split < kSmallItems &&
           2 * (int64_t)max_kv_len <= kSmallSlots * split && parts(split / 2) <= kSmallParts)
      split /= 2;
  }
  if (const int64_t forced = split_override()) split = forced;
  DecodePlan p;
  p.split_tokens = (int32_t)split;
  p.max_splits = (int32_t)((max_kv_len + split - 1) / split);
  if (p.max_splits < 1) p.max_splits = 1;
  return p;
}

size_t decode_workspace_bytes(int32_t B, int32_t hq, const DecodePlan &plan) {
  const size_t parts = (size_t)B * hq * plan.max_splits;
  return parts * (kHeadDim + 2) * sizeof(float);
}

int32_t prefix_slots(const DecodePlan &plan, int32_t max_prefix_len) {
  return (int32_t)((max(max_prefix_len, 0) + (int64_t)plan.split_tokens - 1) / plan.split_tokens);
}

size_t shared_prefix_workspace_bytes(int32_t B, int32_t hq, const DecodePlan &plan,
                                     int32_t max_prefix_len) {
  const size_t parts = (size_t)B * hq * (plan.max_splits + prefix_slots(plan, max_prefix_len));
  return parts * (kHeadDim + 2) * sizeof(float);
}

hipError_t launch_decode(const uint16_t *q, const PagedKV &kv, const int32_t *kv_lens, int32_t B,
                         int32_t hq, int32_t max_kv_len, float scale, float *out, float *lse,
                         void *workspace, const DecodePlan &plan, hipStream_t stream) {
  const DecodeArgs a =
      make_decode_args(q, kv, kv_lens, B, hq, max_kv_len, scale, workspace, plan.max_splits, plan);
  // the G query heads of a KV head are the columns of one 16-column tile, or
  // of two for groups of 17 to 32 heads
  const dim3 grid(kv.hkv, plan.max_splits, B);
  const bool direct = plan.max_splits == 1;
  if (a.group > 16 && direct)
    launch_split<2, true>(kv.fp8, grid, a, out, lse, stream);
  else if (a.group > 16)
    launch_split<2, false>(kv.fp8, grid, a, out, lse, stream);
  else if (direct)
    launch_split<1, true>(kv.fp8, grid, a, out, lse, stream);
  else
    launch_split<1, false>(kv.fp8, grid, a, out, lse, stream);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || direct) return e;
  launch_combine(a, B, out, lse, stream);
  return hipGetLastError();
}

SharedPrefixShape shared_prefix_shape(int32_t group, int32_t num_groups, int32_t max_group_rows,
                                      const DecodePlan &plan, int32_t max_prefix_len) {
  SharedPrefixShape sh;
  // as many rows per prefix chunk as fill the row items' tiles (one tile,
  // two for groups of 17 to 32 heads), so that both kinds of item share one
  // register and LDS budget
  sh.tiles = group > 16 ? 2 : 1;
  sh.rows_per_chunk = max(1, min(max_group_rows, 16 * sh.tiles / group));
  sh.chunks = (max_group_rows + sh.rows_per_chunk - 1) / sh.rows_per_chunk;
  sh.prefix_items = (int64_t)num_groups * sh.chunks * prefix_slots(plan, max_prefix_len);
  sh.prefix_planes = (sh.prefix_items + plan.max_splits - 1) / plan.max_splits;
  sh.row_z = (int64_t)num_groups * max_group_rows;
  return sh;
}

hipError_t launch_decode_shared_prefix(const uint16_t *q, const PagedKV &kv,
                                       const int32_t *kv_lens, const int32_t *group_start,
                                       const int32_t *prefix_len, int32_t B, int32_t hq,
                                       int32_t num_groups, int32_t max_group_rows,
                                       int32_t max_prefix_len, int32_t max_kv_len, float scale,
                                       float *out, float *lse, void *workspace,
                                       const DecodePlan &plan, hipStream_t stream) {
  const int32_t ps = prefix_slots(plan, max_prefix_len);
  DecodeArgs a = make_decode_args(q, kv, kv_lens, B, hq, max_kv_len, scale, workspace,
                           plan.max_splits + ps, plan);
  const SharedPrefixShape sh =
      shared_prefix_shape(a.group, num_groups, max_group_rows, plan, max_prefix_len);
  a.group_start = group_start;
  a.prefix_len = prefix_len;
  a.prefix_slots = ps;
  a.rows_per_chunk = sh.rows_per_chunk;
  a.zdiv = max_group_rows;
  const dim3 grid(kv.hkv, plan.max_splits, (unsigned)(sh.prefix_planes + sh.row_z));
  if (sh.tiles == 2)
    launch_shared<2>(kv.fp8, grid, a, sh, stream);
  else
    launch_shared<1>(kv.fp8, grid, a, sh, stream);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  launch_combine(a, (unsigned)sh.row_z, out, lse, stream);
  return hipGetLastError();
}

}  // namespace ra
