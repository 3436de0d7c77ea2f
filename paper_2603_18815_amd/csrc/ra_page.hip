// Page write and page gather between packed token-major K/V rows and the
// paged pools (K pages token-major [16][128], V pages dim-major [128][16]).
// One workgroup moves one (row, page, KV head) block per pool; V goes through
// LDS so that both sides are accessed in 8- or 16-byte pieces per lane.
// bf16 pools: bit copies. fp8 pools: the write quantizes each bf16 element to
// its E4M3 code (x * fp32(1 / scale), round to nearest even, saturated; the
// block code is shared with the fused append launch), the gather copies the
// codes out.
#include "ra_device.h"
#include "ra_internal.h"
#include "ra_page_write.h"

namespace ra {
namespace {

constexpr int kThreads = 256;
constexpr int kVPitch = kHeadDim + 8;  // LDS row pitch (elements) of the staged V slots

// One page and kHeads KV heads (y) per workgroup. kSearch: the pages are items
// counted by tokens (x, then z), whose row is found by search; otherwise the
// grid is every row (z) at the longest chunk's pages (x).
template <bool kFp8, bool kRope, int kHeads, bool kSearch>
__global__ __launch_bounds__(pwrite::kItemThreads) void page_write_kernel(pwrite::WriteArgs a,
                                                                          int32_t B) {
  __shared__ uint16_t sv[kHeads][kPage][pwrite::kVPitch];
  const pwrite::WriteItem it =
      kSearch ? pwrite::item_page(a, B, (int)(blockIdx.z * gridDim.x + blockIdx.x))
              : pwrite::write_item(a, blockIdx.x, blockIdx.z);
  if (!it.active) return;
  pwrite::write_heads<kFp8, kRope, kHeads>(a, it, blockIdx.y * kHeads, threadIdx.x, sv);
}

template <int kHeads, bool kSearch>
void launch_write(const pwrite::WriteArgs &a, int32_t B, dim3 grid, hipStream_t stream) {
  const dim3 block(pwrite::kItemThreads);
  if (a.fp8 && a.cos_sin)
    hipLaunchKernelGGL((page_write_kernel<true, true, 1, kSearch>), grid, block, 0, stream, a, B);
  else if (a.cos_sin)
    hipLaunchKernelGGL((page_write_kernel<false, true, kHeads, kSearch>), grid, block, 0, stream, a, B);
  else if (a.fp8)
    hipLaunchKernelGGL((page_write_kernel<true, false, 1, kSearch>), grid, block, 0, stream, a, B);
  else
    hipLaunchKernelGGL((page_write_kernel<false, false, 1, kSearch>), grid, block, 0, stream, a, B);
}

// What the two decisions below turn on, measured (kernel time, GB/s of what is
// read and written; 8 KV heads): a page write moves 5.8 to 6.1 TB/s either way
// when its rows are alike.
// - 32 chunks of 64..2,048 tokens: 46.1 us with the full grid (2.0 workgroups
//   per page in use), 48.5 us by search; 54 single tokens and 10 chunks of
//   128..4,096: 44 us with the full grid (10 per page), 23.3 us by search. The
//   grid is searched once it would be over four times the items.
// - Rotated keys: four heads of a page share the cosines and sines, 54 -> 47 us
//   for 32 chunks of 64..2,048 tokens into bf16 pools; one head per workgroup otherwise
//   and for small calls (64 single tokens: 3.9 us with one head, 5.0 us with four; 512
//   chunks of 16: 20.3 and 22.4 us), counted by the pages that their tokens fill, where
//   four leave a remainder (9 heads: 29.2 and 30.9 us) and for fp8 pools (8 chunks of
//   2,048: 21.5 and 21.8 us).
constexpr int kFullGrid = 4;
constexpr int kRopeHeads = 4;
constexpr int64_t kRopeUnits = 8192;   // (full page, head) units from which rotated writes share them

__global__ __launch_bounds__(kThreads) void page_gather_kernel(
    const uint16_t *__restrict__ k_pool, const uint16_t *__restrict__ v_pool,
    const int32_t *__restrict__ block_table, int bt_stride, int num_pages, int hkv,
    const int32_t *__restrict__ lens, const int32_t *__restrict__ cu_out, int total, int max_len,
    uint16_t *__restrict__ k_out, uint16_t *__restrict__ v_out) {
  const int pg = blockIdx.x, g = blockIdx.y, b = blockIdx.z;
  const int tid = threadIdx.x;
  const int cu0 = min(max(cu_out[b], 0), total);
  const int L = min(min(max(lens[b], 0), max_len), total - cu0);
  if (pg * kPage >= L) return;
  const int id = clamp_page(block_table[(size_t)b * bt_stride + pg], num_pages);

  __shared__ uint16_t sv[kPage][kVPitch];
  {
    const int d = tid >> 1, s0 = (tid & 1) * 8;
    const u32x4 w = load_u32x4(v_pool + (((size_t)id * hkv + g) * kHeadDim + d) * kPage + s0);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      sv[s0 + 2 * e][d] = (uint16_t)(w[e] & 0xffffu);
      sv[s0 + 2 * e + 1][d] = (uint16_t)(w[e] >> 16);
    }
  }
  __syncthreads();
  const int slot = tid >> 4, ch = tid & 15;
  const int pos = pg * kPage + slot;
  if (pos < L) {
    const size_t dst = ((size_t)(cu0 + pos) * hkv + g) * kHeadDim + ch * 8;
    const size_t src = (((size_t)id * hkv + g) * kPage + slot) * kHeadDim + ch * 8;
    store_u32x4(k_out + dst, load_u32x4(k_pool + src));
    store_u32x4(v_out + dst, *reinterpret_cast<const u32x4 *>(&sv[slot][ch * 8]));
  }
}

__global__ __launch_bounds__(kThreads) void page_gather_fp8_kernel(
    const uint8_t *__restrict__ k_pool, const uint8_t *__restrict__ v_pool,
    const int32_t *__restrict__ block_table, int bt_stride, int num_pages, int hkv,
    const int32_t *__restrict__ lens, const int32_t *__restrict__ cu_out, int total, int max_len,
    uint8_t *__restrict__ k_out, uint8_t *__restrict__ v_out) {
  const int pg = blockIdx.x, g = blockIdx.y, b = blockIdx.z;
  const int tid = threadIdx.x;
  const int cu0 = min(max(cu_out[b], 0), total);
  const int L = min(min(max(lens[b], 0), max_len), total - cu0);
  if (pg * kPage >= L) return;
  const int id = clamp_page(block_table[(size_t)b * bt_stride + pg], num_pages);

  __shared__ uint8_t sv[kPage][kHeadDim + 16];
  {
    const int d = tid >> 1, s0 = (tid & 1) * 8;
    const u32x2 w = *reinterpret_cast<const u32x2 *>(
        v_pool + (((size_t)id * hkv + g) * kHeadDim + d) * kPage + s0);
#pragma unroll
    for (int e = 0; e < 8; ++e) sv[s0 + e][d] = (uint8_t)(w[e >> 2] >> (8 * (e & 3)));
  }
  __syncthreads();
  const int slot = tid >> 4, ch = tid & 15;
  const int pos = pg * kPage + slot;
  if (pos < L) {
    const size_t dst = ((size_t)(cu0 + pos) * hkv + g) * kHeadDim + ch * 8;
    const size_t src = (((size_t)id * hkv + g) * kPage + slot) * kHeadDim + ch * 8;
    *reinterpret_cast<u32x2 *>(k_out + dst) = *reinterpret_cast<const u32x2 *>(k_pool + src);
    *reinterpret_cast<u32x2 *>(v_out + dst) = *reinterpret_cast<const u32x2 *>(&sv[slot][ch * 8]);
  }
}

}  // namespace

hipError_t launch_page_write(const uint16_t *k_new, const uint16_t *v_new, const int32_t *cu_new,
                             const int32_t *start_pos, const PagedKV &kv, int32_t B,
                             int32_t total_new, int32_t max_new, int32_t max_pos,
                             hipStream_t stream, const float *cos_sin, int32_t rope_rows) {
  // a run of n tokens touches at most (n - 1) / 16 + 2 pages
  const int64_t per_row = ((int64_t)max_new + kPage - 1) / kPage + 1;
  const int64_t counted = pwrite::write_items(B, total_new), row = 1 << 22;   // grid x limit
  const bool search = per_row * B > kFullGrid * counted;
  const int64_t items = search ? counted : per_row * B;
  const bool share = cos_sin && !kv.fp8 && kv.hkv % kRopeHeads == 0 &&
                     (int64_t)(total_new / kPage) * kv.hkv >= kRopeUnits;
  const int heads = share ? kRopeHeads : 1;
  const unsigned groups = (kv.hkv + heads - 1) / heads;
  const dim3 grid = search ? dim3((unsigned)(items < row ? items : row), groups,
                                  (unsigned)((items + row - 1) / row))
                           : dim3((unsigned)per_row, groups, B);
  const pwrite::WriteArgs a = pwrite::write_args(k_new, v_new, cu_new, start_pos, kv, total_new,
                                                 max_new, max_pos, cos_sin, rope_rows);
  if (search && heads > 1)
    launch_write<kRopeHeads, true>(a, B, grid, stream);
  else if (search)
    launch_write<1, true>(a, B, grid, stream);
  else if (heads > 1)
    launch_write<kRopeHeads, false>(a, B, grid, stream);
  else
    launch_write<1, false>(a, B, grid, stream);
  return hipGetLastError();
}

hipError_t launch_page_gather(const PagedKV &kv, const int32_t *lens, const int32_t *cu_out,
                              int32_t B, int32_t total, int32_t max_len, uint16_t *k_out,
                              uint16_t *v_out, hipStream_t stream) {
  const dim3 grid((unsigned)(((int64_t)max_len + kPage - 1) / kPage), kv.hkv, B);
  if (kv.fp8)
    hipLaunchKernelGGL(page_gather_fp8_kernel, grid, dim3(kThreads), 0, stream,
                       reinterpret_cast<const uint8_t *>(kv.k_pool),
                       reinterpret_cast<const uint8_t *>(kv.v_pool), kv.block_table, kv.bt_stride,
                       kv.num_pages, kv.hkv, lens, cu_out, total, max_len,
                       reinterpret_cast<uint8_t *>(k_out), reinterpret_cast<uint8_t *>(v_out));
  else
    hipLaunchKernelGGL(page_gather_kernel, grid, dim3(kThreads), 0, stream, kv.k_pool, kv.v_pool,
                       kv.block_table, kv.bt_stride, kv.num_pages, kv.hkv, lens, cu_out, total,
                       max_len, k_out, v_out);
  return hipGetLastError();
}

}  // namespace ra
