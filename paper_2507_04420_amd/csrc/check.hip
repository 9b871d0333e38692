// Device-side verification of a mate array (the product's own check; the
// test suite pins it against the independent CPU checker).
//
// Counts, per class, the ways a mate array can fail to be a maximal matching
// of the graph (Section II-B): a mate out of range, a vertex matched to
// itself, an asymmetric pair, a pair that is not an edge, and an edge whose
// two endpoints are both unmatched.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstring>

#include "batch.h"
#include "internal.h"
#include "mm.h"

using mmi::fail;
#define HIP_TRY MMI_HIP_TRY

namespace {

// Lists longer than this are checked by the whole wavefront, one after the
// other; those up to it are laid end to end (scan_lists), which fills every step
// whatever their lengths but reads them to their ends, where a list by itself
// is left at its key. Beyond a step and a half of entries the latter is worth more:
// with the line at 2048 and at 384, the call, a clique of 2000 vertices 368 and 109 us
// (a lane a list: 266), of 390 84 and 50, ER of 20000 vertices and 1024 entries each
// 168 and 84; lists of about 256 are the same either way, but with the line there
// ER of 65536 and 256, all unmatched, took 116 against 110. It also bounds the
// laid-out length of a wavefront's 64 lists.
constexpr int64_t kFlatList = 384;
// A matched vertex whose list is longer than this leaves the search for its
// edge to its mate when the mate's list is shorter.
constexpr int64_t kOwnList = 32;
// Entries of a graph whose vertices are checked by a lane each (check_alone): all
// that 64 vertices can have without duplicates.
constexpr int64_t kAlone = 64 * 64;
// Single graphs of at least kBitsFrom vertices and kBitsDegree entries per
// vertex get a bit per vertex for the scans of unmatched vertices: on a skewed
// graph a quarter of the vertices stay unmatched, and every entry of theirs is
// a random access, to a line of a mate array far larger than the 4 MB of an
// XCD's L2, or to a bit of an array that fits it. The bits cost a pass over the
// mates and an allocation (15 to 25 us), so below 2^23 vertices or on sparse
// graphs, whose scans are few or local, they do not pay or not always. The call
// without and with them: R-MAT-25 951 and 671 us, R-MAT-24 460 and 373, ER of
// 2^24 vertices and 8 entries each 409 and 382, of 2^22 and 16 131 and 128; but a mesh
// of 1e7 96 and 118.
constexpr int64_t kBitsFrom = (int64_t)1 << 23;
constexpr int64_t kBitsDegree = 8;
constexpr int kThreads = 1024;
constexpr int kWindow = 256;  // laid-out entries a wavefront takes per step, four a lane

// Loads are typed as global ones. Through generic pointers (a batch's graphs
// keep theirs in memory, a list's place comes from LDS) they would count as LDS
// operations too, and every LDS read would wait for the loads before it.
template <typename T>
using Global = const __attribute__((address_space(1))) T*;

// An id is read once; with BITS it must not push the bits out of L2 (the call,
// R-MAT-25 685 -> 671 us, R-MAT-24 unchanged; offsets read so as well took
// R-MAT-25 to 655 and R-MAT-24 from 372 to 389).
template <bool BITS>
__device__ __forceinline__ int32_t load_id(Global<int32_t> p) {
  return BITS ? __builtin_nontemporal_load(p) : *p;
}

// What the lists of a call lead to, the same for all lanes.
struct Ids {
  Global<int32_t> nbr;
  Global<uint32_t> free;  // mates, or (BITS) a bit per vertex, set if unmatched
  uint32_t n;             // vertices
};

// One list to examine: for key >= 0, whether it holds key; else, the list of the
// unmatched vertex ~key, how many of its entries lead to other unmatched vertices.
struct alignas(16) List {
  int64_t first;  // its first entry; laid end to end: less its first position
  int32_t key;
};

// One wavefront's LDS.
struct WaveLds {
  List list[64];
  uint32_t head[kWindow / 4];  // byte p: a list starts at position p of the window
  uint8_t found[64];
};

__device__ __forceinline__ uint32_t lanes_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                   __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Of four entries a lane, how many lead to an unmatched vertex; only those with
// look[q] (which have an id in range) are read, all of them before the first is
// looked at.
template <bool BITS>
__device__ __forceinline__ uint32_t unmatched(Global<uint32_t> free, const int32_t id[4],
                                              const bool look[4]) {
  uint32_t v[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    v[q] = 0;
    if (look[q]) v[q] = free[BITS ? (uint32_t)id[q] >> 5 : (uint32_t)id[q]];
  }
  uint32_t sum = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) sum += BITS ? (v[q] >> (id[q] & 31)) & 1u : (uint32_t)(v[q] == ~0u);
  return sum;
}

// LDS written by one lane is read by another lane of the same wavefront.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Examines one list per lane (len <= 0: none) with the whole wavefront.
// Returns whether this lane's list holds its key; adds the uncovered entries of
// the others to *uncovered.
//
// The lists are laid end to end and taken kWindow entries at a time: every
// lane reads four ids, then the four mates those lead to, whatever the lists'
// lengths, so that a long list does not hold the other 63 lanes and the loads
// of a step are independent. The list an entry belongs to is the count of
// list starts up to it: starts are marked in LDS and counted with a ballot.
//
// With few entries per vertex its instructions bound it, on large graphs the
// random reads. What describes the call (Ids) is the same for all lanes and
// stays in scalar registers, a list is one 16-byte LDS read, the loads of a
// step are all issued before the first is waited for, and the kernels fit 64
// vector registers without spilling any, so two workgroups share a CU. Against a list that
// names its graph and generic pointers, the call: a mesh of 1e7 vertices
// 120 -> 96 us, ER of 2^22 vertices and 16 entries each 136 -> 131, R-MAT-25 683 -> 671;
// with two registers spilled ER took 158.
template <bool BITS>
__device__ __forceinline__ bool scan_lists(const Ids& g, const List& mine, int64_t len, WaveLds& w,
                                           int32_t* uncovered) {
  const int lane = (int)(threadIdx.x & 63);
  const bool flat = len > 0 && len <= kFlatList;
  const uint64_t fm = __ballot(flat);
  bool hit = false;
  if (fm) {
    // inclusive prefix sum of the flat lists' lengths
    int32_t sum = flat ? (int32_t)len : 0;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int32_t o = __shfl_up(sum, d, 64);
      if (lane >= d) sum += o;
    }
    const int32_t total = __builtin_amdgcn_readlane(sum, 63);
    const int32_t start = sum - (flat ? (int32_t)len : 0);
    const uint32_t slot = lanes_below(fm);
    if (flat) {
      w.list[slot] = List{mine.first - start, mine.key};
      w.found[slot] = 0;
    }
    int32_t before = -1;  // lists started before the window, less one
    for (int32_t base = 0; base < total; base += kWindow) {
      w.head[lane] = 0;
      wave_sync();
      if (flat && start >= base && start < base + kWindow)
        reinterpret_cast<uint8_t*>(w.head)[start - base] = 1;
      wave_sync();
      int32_t id[4], at[4];
      List l[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int32_t starts = reinterpret_cast<const uint8_t*>(w.head)[q * 64 + lane];
        const uint64_t h = __ballot(starts != 0);
        at[q] = before + starts + (int32_t)lanes_below(h);
        before += (int32_t)__popcll(h);
        l[q] = w.list[at[q]];
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int32_t pos = base + q * 64 + lane;
        id[q] = -1;
        if (pos < total) id[q] = load_id<BITS>(g.nbr + (l[q].first + pos));
      }
      wave_sync();
      bool look[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const bool in = (uint32_t)id[q] < g.n;
        if (in && id[q] == l[q].key) w.found[at[q]] = 1;
        look[q] = in && l[q].key < 0 && id[q] != ~l[q].key;
      }
      *uncovered += (int32_t)unmatched<BITS>(g.free, id, look);
    }
    wave_sync();
    hit = flat && w.found[slot] != 0;
    wave_sync();
  }
  uint64_t longs = __ballot(len > kFlatList);
  while (longs) {
    const int src = __builtin_ctzll(longs);
    longs &= longs - 1;
    const int64_t first = __shfl((long long)mine.first, src, 64);
    const int64_t m = __shfl((long long)len, src, 64);
    const int32_t key = __shfl(mine.key, src, 64);
    bool any = false;
    for (int64_t i = 0; i < m && !any; i += kWindow) {
      int32_t id[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        id[q] = -1;
        if (i + q * 64 + lane < m) id[q] = load_id<BITS>(g.nbr + (first + i + q * 64 + lane));
      }
      if (key >= 0) {
        any = __ballot(id[0] == key || id[1] == key || id[2] == key || id[3] == key) != 0;
      } else {
        bool look[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) look[q] = (uint32_t)id[q] < g.n && id[q] != ~key;
        *uncovered += (int32_t)unmatched<BITS>(g.free, id, look);
      }
    }
    if (lane == src) hit = any;
  }
  return hit;
}

// Counts are 32 bits a lane (c[2] may be negative in between): the entries a lane
// looks at are a 64th of its wavefront's, and 288 GB hold 7.2e10.
//
// Checks 64 vertices, one per lane (valid: the lane has one): vertex x of a
// graph of n vertices whose offsets, ids and mates are based at its first
// vertex; free: the mates again, or (BITS) its bits of unmatched vertices.
//
// mate[mate[x]] == x is read (a random access) by the lower end only: counting
// every matched vertex as asymmetric and taking two off for each mutual pair
// leaves the vertices whose mate does not name them.
//
// A pair's edge may be in either end's list. An end with a short list searches
// its own, which is read coalesced with its neighbours in the block; an end
// with a long list leaves the search to its mate if that has the shorter one
// (the search of a hub's list for one id would read most of it), and the end
// that searches counts for both. An edge not found there is searched in the
// other list (one-sided input).
template <typename OffT, bool BITS>
__device__ __forceinline__ void check_vertices(const OffT* offsets, const int32_t* nbr, int64_t n,
                                               const int32_t* mates, const void* free, int64_t x,
                                               bool valid, WaveLds& w, int32_t c[6]) {
  const Global<OffT> off = (Global<OffT>)offsets;
  const Global<int32_t> mate = (Global<int32_t>)mates;
  const Ids g{(Global<int32_t>)nbr, (Global<uint32_t>)free, (uint32_t)n};
  List l{0, ~(int32_t)x};
  int64_t len = 0;
  unsigned weight = 1;
  bool search = false;
  if (valid) {
    const int64_t y = mate[x];
    const int64_t b = (int64_t)off[x], e = (int64_t)off[x + 1];
    if (y < -1 || y >= n) {
      ++c[0];
    } else if (y == x) {
      ++c[1];
      ++c[5];
    } else if (y >= 0) {
      ++c[5];
      ++c[2];
      const bool longl = e - b > kOwnList;
      const bool mutual = (x < y || longl) && (int64_t)mate[y] == x;
      if (mutual && x < y) c[2] -= 2;
      search = true;
      if (mutual && longl) {
        const int64_t ly = (int64_t)off[y + 1] - (int64_t)off[y];
        if (ly <= kOwnList || ly < e - b || (ly == e - b && y < x))
          search = false;
        else
          weight = 2;  // the mate's list is longer: it leaves the search to this end
      }
      l.key = (int32_t)y;
    }
    if (search || y == -1) {
      l.first = b;
      len = e - b;
    }
  }
  bool hit = scan_lists<BITS>(g, l, len, w, &c[4]);
  const bool again = search && !hit;
  if (!__ballot(again)) return;
  len = 0;
  if (again) {
    const int64_t y = l.key, b = (int64_t)off[y], e = (int64_t)off[y + 1];
    // a mate with a long list has left the search to this end
    if (weight == 1 && e - b > kOwnList && (int64_t)mate[y] == x) weight = 2;
    l.key = (int32_t)x;
    l.first = b;
    len = e - b;
  }
  hit = scan_lists<BITS>(g, l, len, w, &c[4]);
  if (again && !hit) c[3] += (int32_t)weight;
}

// Sums the block's counts and adds them to out, one atomic per nonzero count
// and block: atomics of all blocks on the same six words are done one after
// the other, about 12 ns each.
__device__ __forceinline__ void flush_counts(int32_t c[6], unsigned long long* out) {
  __shared__ unsigned long long part[kThreads / 64][6];
  const int lane = (int)(threadIdx.x & 63);
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    unsigned long long s = (unsigned long long)(long long)c[k];
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) s += __shfl_xor(s, d, 64);
    if (lane == 0) part[threadIdx.x >> 6][k] = s;
  }
  __syncthreads();
  if (threadIdx.x < 6) {
    unsigned long long s = 0;
    for (int q = 0; q < (int)(blockDim.x >> 6); ++q) s += part[q][threadIdx.x];
    if (s)
      __hip_atomic_fetch_add(out + threadIdx.x, s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// One bit per vertex, set if it is unmatched.
__global__ void free_bits_kernel(const int32_t* __restrict__ mate, int64_t n,
                                 uint64_t* __restrict__ bits) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int lane = (int)(threadIdx.x & 63);
  for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x - lane < n; x += stride) {
    const uint64_t m = __ballot(x < n && mate[x] == -1);
    if (lane == 0) bits[x >> 6] = m;
  }
}

template <typename OffT, bool BITS>
__global__ __launch_bounds__(kThreads) void check_kernel(
    const OffT* __restrict__ off, const int32_t* __restrict__ nbr, int64_t n,
    const int32_t* __restrict__ mate, const void* __restrict__ free, unsigned long long* out) {
  __shared__ WaveLds lds[kThreads / 64];
  int32_t c[6] = {0, 0, 0, 0, 0, 0};
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
       x - (int64_t)(threadIdx.x & 63) < n; x += stride)
    check_vertices<OffT, BITS>(off, nbr, n, mate, free, x, x < n, lds[threadIdx.x >> 6], c);
  flush_counts(c, out);
}

// The graph of global vertex v: the last one in [lo, hi) that starts at or
// before it.
__device__ __forceinline__ int graph_of(const int64_t* vtx_off, int lo, int hi, int64_t v) {
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (vtx_off[mid] <= v) lo = mid; else hi = mid;
  }
  return lo;
}

// The same where the graph is lo or one of the next few.
__device__ __forceinline__ int graph_from(const int64_t* vtx_off, int lo, int hi, int64_t v) {
  int64_t at = lo, step = 1;
  while (at + step < hi && vtx_off[at + step] <= v) {
    at += step;
    step *= 2;
  }
  return graph_of(vtx_off, (int)at, (int)(at + step < hi ? at + step : hi), v);
}

// One vertex of a small graph, checked by its lane alone.
__device__ __forceinline__ void check_alone(const mmb::GraphDesc& d, const int32_t* mates, int64_t x,
                                            int32_t c[6]) {
  const Global<int64_t> off = (Global<int64_t>)d.off;
  const Global<int32_t> nbr = (Global<int32_t>)d.nbr;
  const Global<int32_t> mate = (Global<int32_t>)mates;
  const int64_t y = mate[x];
  int64_t b = off[x], e = off[x + 1];
  if (y < -1 || y >= d.n) {
    ++c[0];
  } else if (y == x) {
    ++c[1];
    ++c[5];
  } else if (y >= 0) {
    bool edge = false;
    for (; b < e && !edge; ++b) edge = nbr[b] == y;
    if (!edge) {
      b = off[y];
      e = off[y + 1];
      for (; b < e && !edge; ++b) edge = nbr[b] == x;
    }
    ++c[5];
    c[2] += mate[y] != x;
    c[3] += !edge;
  } else {
    for (; b < e; ++b) {
      const int64_t z = nbr[b];
      if (z >= 0 && z < d.n && z != x) c[4] += mate[z] == -1;
    }
  }
}

// A batch: 64 consecutive vertices lie in one graph unless it ends among them.
// The wavefront takes the lanes of one graph at a time, so that the search for
// it and what describes it stay in scalar registers: with a graph per lane the
// kernel took 73 registers, of which one workgroup of 16 wavefronts fits a CU
// (267 us for 256 graphs of 8.5e6 vertices in all; two fit now, 175 us, and 152 with
// the loads of scan_lists as they are; 1024 small graphs 151 and 131 us with the
// call around it).
//
// CROWDED: some 64 consecutive vertices may belong to more than kCrowd graphs. One
// graph after the other would then leave most lanes idle, so the lanes of such a
// wavefront look up their own graphs and check alone the vertices of those that
// lie within it whole (check_vertices counts for both ends of a pair, so a graph
// goes one way or the other) and have at most kAlone entries; the others go on
// as above. The call without and with it: 1e6 graphs of 1 to 8 vertices 917 and 169
// us, 5e5 of one vertex 366 and 45, 1e5 of 1 to 16 130 and 77; of 8 to 16, seldom
// as crowded, 117 and 84, which is the search that starts at the graph before.
template <bool CROWDED>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(8))) void check_batch_kernel(
    const mmb::GraphDesc* __restrict__ descs, const int64_t* __restrict__ vtx_off,
    int32_t num_graphs, const int32_t* __restrict__ mate, unsigned long long* out) {
  __shared__ WaveLds lds[kThreads / 64];
  int32_t c[6] = {0, 0, 0, 0, 0, 0};
  const int64_t N = vtx_off[num_graphs];
  const int lane = (int)(threadIdx.x & 63);
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v - lane < N; v += stride) {
    // wavefront-uniform: the search runs in scalar registers
    const int64_t first = ((int64_t)__builtin_amdgcn_readfirstlane((int)((v - lane) >> 32)) << 32) |
                          (uint32_t)__builtin_amdgcn_readfirstlane((int)(v - lane));
    uint64_t todo = __ballot(v < N);
    int g = graph_of(vtx_off, 0, num_graphs, first);
    if (CROWDED && g + mmb::kCrowd <= num_graphs && vtx_off[g + mmb::kCrowd] < first + 64) {
      bool done = false;
      if (v < N) {
        const mmb::GraphDesc& d = descs[graph_from(vtx_off, g, num_graphs, v)];
        done = d.v0 >= first && d.v0 + d.n <= first + 64 && d.off[d.n] - d.off[0] <= kAlone;
        if (done) check_alone(d, mate + d.v0, v - d.v0, c);
      }
      todo &= ~__ballot(done);
      if (todo) g = graph_from(vtx_off, g, num_graphs, first + __builtin_ctzll(todo));
    }
    while (todo) {
      const mmb::GraphDesc& d = descs[g];
      const int32_t* m = mate + d.v0;
      const bool mine = ((todo >> lane) & 1) && v - d.v0 < d.n;
      check_vertices<int64_t, false>(d.off, d.nbr, d.n, m, m, v - d.v0, mine, lds[threadIdx.x >> 6], c);
      todo &= ~__ballot(mine);
      if (todo) g = graph_from(vtx_off, g + 1, num_graphs, first + __builtin_ctzll(todo));
    }
  }
  flush_counts(c, out);
}

mm_status finish(unsigned long long* dev, hipStream_t s, int64_t* counts) {
  unsigned long long h[6];
  HIP_TRY(mmi::read_back(h, dev, sizeof(h), s));
  for (int k = 0; k < 6; ++k) counts[k] = (int64_t)h[k];
  return MM_OK;
}

// At most 512 workgroups (two of 16 wavefronts fill a CU), so that few of them
// add to the counts at the end; a graph too small for 512 large ones gets
// smaller ones, down to a wavefront each, to be spread over all CUs.
struct Grid {
  unsigned blocks, threads;
};
Grid grid_of(int64_t n) {
  int64_t t = 64;
  while (t < kThreads && n > 512 * t) t *= 2;
  const int64_t b = (n + t - 1) / t;
  return Grid{(unsigned)(b > 512 ? 512 : b), (unsigned)t};
}

template <typename OffT>
void launch_check(const Grid& gr, const OffT* off, const int32_t* nbr, int64_t n, const int32_t* mate,
                  const uint64_t* bits, unsigned long long* dev, hipStream_t s) {
  if (bits)
    hipLaunchKernelGGL((check_kernel<OffT, true>), dim3(gr.blocks), dim3(gr.threads), 0, s, off, nbr,
                       n, mate, bits, dev);
  else
    hipLaunchKernelGGL((check_kernel<OffT, false>), dim3(gr.blocks), dim3(gr.threads), 0, s, off, nbr,
                       n, mate, mate, dev);
}

}  // namespace

extern "C" {

mm_status mm_check(mm_handle h, void* stream, const int32_t* match, int64_t* counts) {
  if (!h || !counts || (!match && mmi::handle_n(h) > 0))
    return fail(MM_ERR_INVALID_ARG, "null argument");
  hipStream_t s = static_cast<hipStream_t>(stream);
  unsigned long long* dev = reinterpret_cast<unsigned long long*>(mmi::handle_ws(h) + mmi::kCheckOffset);
  HIP_TRY(hipMemsetAsync(dev, 0, 6 * sizeof(unsigned long long), s));
  const int64_t n = mmi::handle_n(h);
  if (n > 0) {
    const Grid gr = grid_of(n);
    uint64_t* bits = nullptr;
    if (n >= kBitsFrom && mmi::handle_m(h) / n >= kBitsDegree &&
        hipMallocAsync(reinterpret_cast<void**>(&bits), (size_t)((n + 63) / 64) * 8, s) != hipSuccess) {
      bits = nullptr;  // no memory for them: the mates themselves are read
      (void)hipGetLastError();
    }
    if (bits)
      hipLaunchKernelGGL(free_bits_kernel, dim3(2048), dim3(256), 0, s, match, n, bits);
    if (mmi::handle_off64(h))
      launch_check(gr, static_cast<const int64_t*>(mmi::handle_off(h)), mmi::handle_nbr(h), n, match,
                   bits, dev, s);
    else
      launch_check(gr, static_cast<const int32_t*>(mmi::handle_off(h)), mmi::handle_nbr(h), n, match,
                   bits, dev, s);
    const hipError_t e = hipGetLastError();
    if (bits) (void)hipFreeAsync(bits, s);
    HIP_TRY(e);
  }
  return finish(dev, s, counts);
}

mm_status mm_batch_check(mm_batch_handle b, void* stream, const int32_t* match, int64_t* counts) {
  if (!b || !counts) return fail(MM_ERR_INVALID_ARG, "null argument");
  hipStream_t s = static_cast<hipStream_t>(stream);
  const mmb::BatchInfo info = mmb::batch_info(b);
  if (!match && info.N > 0) return fail(MM_ERR_INVALID_ARG, "match is null");
  unsigned long long* dev = reinterpret_cast<unsigned long long*>(info.ws + mmi::kCheckOffset);
  HIP_TRY(hipMemsetAsync(dev, 0, 6 * sizeof(unsigned long long), s));
  if (info.N > 0) {
    const Grid gr = grid_of(info.N);
    const auto kernel = info.crowded ? check_batch_kernel<true> : check_batch_kernel<false>;
    hipLaunchKernelGGL(kernel, dim3(gr.blocks), dim3(gr.threads), 0, s, info.descs, info.vtx_off,
                       info.G, match, dev);
    HIP_TRY(hipGetLastError());
  }
  return finish(dev, s, counts);
}

}  // extern "C"
