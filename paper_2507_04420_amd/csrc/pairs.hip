// Matched-pair list output (the `matches` array that Algorithm 1 fills and returns).
//
// The sweep records its result in the mate array; this pass turns a mate
// array into the list of matched pairs (u, v), u < v, each pair once. A
// workgroup compacts a tile of vertices and reserves its slots with one atomic
// add on a shared cursor, the GPU form of the paper's per-thread buffers taken
// from one shared block. The order of the pairs is not specified.
//
// Bound: the mates are read and the pairs written once (56 MB for 8e6 vertices
// of which 80% are matched, 12 us at the rate of a large copy); what costs is
// the cursor, since adds to one word are done one after the other, 12 ns each
// whatever adds them. An add per wavefront and 64 vertices took 1474 us there;
// with 8192 vertices per add the adds are 977, under the loads of other tiles,
// and the kernel takes 24 us.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "internal.h"
#include "mm.h"

using mmi::fail;
#define HIP_TRY MMI_HIP_TRY

namespace {

constexpr size_t kPairsCursorOffset = mmi::kCheckOffset + 64;

constexpr int kThreads = 256;

// A tile is kThreads * ROWS vertices, a wavefront's part of it 64 * ROWS
// consecutive ones, ROWS per lane.
template <int ROWS>
__global__ __launch_bounds__(kThreads) void pairs_kernel(const int32_t* __restrict__ mate, int64_t n,
                                                         int32_t* __restrict__ out, int64_t cap,
                                                         unsigned long long* cursor) {
  constexpr int kWaves = kThreads / 64;
  __shared__ uint32_t count[2][kWaves];
  __shared__ unsigned long long first[2];
  const int lane = (int)(threadIdx.x & 63), wave = (int)(threadIdx.x >> 6);
  const int64_t tile = (int64_t)kThreads * ROWS;
  int odd = 0;  // two sets of LDS words, so that a tile needs no barrier before it
  for (int64_t t = (int64_t)blockIdx.x * tile; t < n; t += (int64_t)gridDim.x * tile, odd ^= 1) {
    const int64_t base = t + (int64_t)wave * 64 * ROWS + lane;
    int32_t y[ROWS];
    uint64_t lead[ROWS];  // the lower end of a pair writes it
    uint32_t mine = 0;
#pragma unroll
    for (int r = 0; r < ROWS; ++r) y[r] = base + r * 64 < n ? mate[base + r * 64] : -1;
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
      lead[r] = __ballot((int64_t)y[r] > base + r * 64 && (int64_t)y[r] < n);
      mine += (uint32_t)__popcll(lead[r]);
    }
    if (lane == 0) count[odd][wave] = mine;
    __syncthreads();
    if (threadIdx.x == 0) {
      uint32_t all = 0;
      for (int w = 0; w < kWaves; ++w) all += count[odd][w];
      first[odd] = all ? __hip_atomic_fetch_add(cursor, (unsigned long long)all, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT)
                       : 0;
    }
    __syncthreads();
    int64_t slot = (int64_t)first[odd];
    for (int w = 0; w < wave; ++w) slot += count[odd][w];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
      if ((lead[r] >> lane) & 1) {
        const int64_t k = slot + __builtin_amdgcn_mbcnt_hi(
                                     (uint32_t)(lead[r] >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)lead[r], 0u));
        if (k < cap) {
          out[2 * k] = (int32_t)(base + r * 64);
          out[2 * k + 1] = y[r];
        }
      }
      slot += (int64_t)__popcll(lead[r]);
    }
  }
}

template <int ROWS>
void launch_pairs(const int32_t* mate, int64_t n, int32_t* out, int64_t cap,
                  unsigned long long* cursor, hipStream_t s) {
  const int64_t tiles = (n + kThreads * ROWS - 1) / (kThreads * ROWS);
  hipLaunchKernelGGL((pairs_kernel<ROWS>), dim3((unsigned)(tiles < 2048 ? tiles : 2048)),
                     dim3(kThreads), 0, s, mate, n, out, cap, cursor);
}

}  // namespace

extern "C" {

mm_status mm_pairs(mm_handle h, void* stream, const int32_t* match, int32_t* pairs, int64_t cap,
                   int64_t* count) {
  if (!h || !count) return fail(MM_ERR_INVALID_ARG, "null argument");
  const int64_t n = mmi::handle_n(h);
  if (!match && n > 0) return fail(MM_ERR_INVALID_ARG, "match is null");
  if (cap < 0 || (!pairs && cap > 0)) return fail(MM_ERR_INVALID_ARG, "bad pairs buffer");
  hipStream_t s = static_cast<hipStream_t>(stream);
  auto* cursor = reinterpret_cast<unsigned long long*>(mmi::handle_ws(h) + kPairsCursorOffset);
  HIP_TRY(hipMemsetAsync(cursor, 0, sizeof(unsigned long long), s));
  if (n > 0) {
    // the adds grow with n / ROWS (12 ns each), the CUs in use with the tiles: 256
    // of them up to 65536 vertices, then 1024 at most up to 2^21, then n / 8192
    if (n <= 65536)
      launch_pairs<1>(match, n, pairs, cap, cursor, s);
    else if (n <= (int64_t)1 << 21)
      launch_pairs<8>(match, n, pairs, cap, cursor, s);
    else
      launch_pairs<32>(match, n, pairs, cap, cursor, s);
    HIP_TRY(hipGetLastError());
  }
  unsigned long long c = 0;
  HIP_TRY(mmi::read_back(&c, cursor, sizeof(c), s));
  *count = (int64_t)c;
  if ((int64_t)c > cap)
    return fail(MM_ERR_OUT_OF_MEMORY, "%lld pairs, buffer holds %lld (only the first %lld written)",
                (long long)c, (long long)cap, (long long)cap);
  return MM_OK;
}

}  // extern "C"
