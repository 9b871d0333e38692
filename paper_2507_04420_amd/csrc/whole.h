// A graph small enough for one wavefront, swept with its states in that
// wavefront's LDS.
//
// When one wavefront sweeps a whole graph (a small batch member, or a small
// graph alone), no other wavefront ever reads or writes that graph's states.
// They can then live in LDS instead of device memory: Algorithm 1's reserve,
// CAS and commit become LDS atomics, whose latency is a small fraction of a
// device-scope atomic's (those pass L2 and go to memory). The protocol is the
// same (Section IV-B, Fig. 4) in its two-phase form (v is reserved like u,
// then both are marked matched): a CAS on a word that holds several vertices
// would fail whenever another lane changed one beside it, while a fetch_or
// reservation never does. State and mate of a vertex share a 16-bit entry (32 KB
// for 16384 vertices), and a last pass writes the whole output, coalesced:
// inside the sweep the only device-memory operations left are the loads of
// offsets and ids, so a loop trip never waits for a store.
//
// The instrumented build, and a multigraph of more than 2^30 entries, run the
// general sweep on states of 2 bits with the mates beside them (LayoutLds), which
// follows the same schedule.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mm.h"
#include "protocol.h"
#include "sweep.h"

namespace mmk {

// LDS words a wavefront needs for n vertices: the states (2 bits each), then
// the mates (16 bits each), each part a whole number of 16-byte quads.
__host__ __device__ __forceinline__ int64_t whole_state_words(int64_t n) {
  return ((n + 15) / 16 + 3) / 4 * 4;
}
__host__ __device__ __forceinline__ int64_t whole_lds_words(int64_t n) {
  return whole_state_words(n) + ((n + 1) / 2 + 3) / 4 * 4;
}

// The loop below keeps state and mate of a vertex in one 16-bit entry.
__host__ __device__ __forceinline__ int64_t whole_entry_words(int64_t n) {
  return ((n + 1) / 2 + 3) / 4 * 4;  // fewer than whole_lds_words(n)
}
static_assert(MM_LDS_WHOLE_MAX <= 1 << 14, "ids of 14 bits beside two state bits");

// The two-phase packed layout with its mates in LDS (16-bit ids: every
// vertex id of such a graph is below MM_LDS_WHOLE_MAX <= 32768).
struct LayoutLds : LayoutPacked<2, true> {
  int16_t* mate16;
  __device__ __forceinline__ void commit(int64_t u, int64_t v) const {
    or_agent(wp(u), 2u << shift(u));
    or_agent(wp(v), 2u << shift(v));
    mate16[u] = (int16_t)v;
    mate16[v] = (int16_t)u;
  }
};
static_assert(MM_LDS_WHOLE_MAX <= 32768, "16-bit mates");

// ---------------------------------------------------------------- the loop
// sweep_block's loop for one wavefront and states in LDS.
//
// What bounds it: the wavefront is alone on its SIMD, so a pass takes its loop
// trips (a few per 64 sources) times the length of a trip, and a trip is as
// long as its instructions plus the waits between them. sweep_block's trip
// takes 1.8 us there: 500 instructions, half of them scalar ones and branches
// around the cases of its switches, and a wait for a load from device memory.
//
// The schedule is sweep_block's, trip by trip: which lane takes which source,
// what every lane does on which trip, and in which order the operations of a
// trip reach LDS (first the reads of lanes waiting for v, then the
// reservations of v, the reads of lanes waiting for u, the reservations of u).
// So is the matching, therefore, to the last mate. What differs is what a trip
// costs:
//   * a state and its mate are one 16-bit entry (mate in bits 0-13, reserved in
//     bit 14, matched in bit 15): the filter reads the entry and looks at its
//     top bit, a commit or a release is one 16-bit store by the holder;
//   * ids and offsets are loaded ahead of the trip that uses them. A lane's
//     sources follow each other in the graph, so the offset of the next one
//     is known a chunk early and its first four ids are in the queue slot
//     that hands it out; while a lane examines four ids, the next four are on
//     their way;
//   * positions are 32 bits wide, relative to the graph's first entry, and a
//     lane's up to four candidates are bit masks instead of loops;
//   * the phases are lane masks in scalar registers, so that what a trip does
//     next is a few mask operations instead of a switch per lane;
//   * the rare cases (waits, assists) are behind one uniform branch each.
// A trip is 300 instructions and 0.8 us: R-MAT-13 (253 trips) 454 -> 205 us,
// ER of 16000 vertices (796 trips) 1426 -> 625 us; a batch of 1024 graphs of up to
// 16384 vertices, one to a SIMD, 2195 -> 861 us.

// Up to this many entries a graph's positions fit the loop's 32 bits with room
// for the reads ahead; a larger one (a multigraph: it has at most 16384
// vertices) takes sweep_block.
constexpr int64_t kWholeEntries = (int64_t)1 << 30;

// LDS entries are read and written as 16-bit values and reserved by 32-bit
// atomics on the word that holds two of them.
typedef uint16_t __attribute__((may_alias)) lds_u16;
typedef uint32_t __attribute__((may_alias)) lds_u32;

// Four ids in one load; a list starts at any entry, so 4-byte alignment.
typedef int32_t ids4 __attribute__((ext_vector_type(4), aligned(4)));

// A wavefront's queue of sources (kQueue slots each): positions, first ids, id.
struct WholeQueue {
  int32_t b[kQueue], e[kQueue];
  ids4 ids[kQueue];
  uint16_t x[kQueue];
  uint16_t ahead[64];  // the ids an assist reads ahead, 0xffff for none
};
static_assert(sizeof(WholeQueue) <= sizeof(QSlot) * kQueue, "shares the QSlot ring's LDS");

// Keeps the compiler from moving LDS accesses across it; the hardware does a
// wavefront's LDS operations in the order they are issued.
__device__ __forceinline__ void lds_order() { asm volatile("" ::: "memory"); }

__device__ __forceinline__ bool in(uint64_t lanes) {
  return __builtin_amdgcn_inverse_ballot_w64(lanes);
}

template <typename OffT, bool UPPER, class GOff, class GNbr>
__device__ __forceinline__ void whole_loop(const SweepParams& a, GOff __restrict__ off,
                                           GNbr __restrict__ nbr, const int32_t n, const int32_t m,
                                           lds_u16* st, WholeQueue& q) {
  constexpr uint32_t kRsv = 0x4000u, kMch = 0x8000u;
  const int lane = (int)(threadIdx.x & 63);
  const int W = a.scan_width;
  const int32_t stride = (n + 63) >> 6;  // chunk c holds the sources lane * stride + c
  const int64_t cap = a.iter_cap > 0 ? a.iter_cap : 65536 + 8 * (int64_t)m;
  const int64_t base = (int64_t)off[0];
  // whose state reads take one candidate: all, those of a source's first read, none
  const uint64_t one_all = a.probe_first == 2 ? ~0ull : 0ull;
  const uint64_t one_first = a.probe_first ? ~0ull : 0ull;
  // whether a lane gives u back while it waits for v
  const uint64_t give_back = a.wait_release ? ~0ull : 0ull;
  const int32_t m4 = m - 4;  // the last position at which four ids can be read
  nbr += base;
  using GIds = const __attribute__((address_space(1))) ids4*;

  auto reserve = [&](int32_t v) -> uint32_t {
    return __hip_atomic_fetch_or(reinterpret_cast<lds_u32*>(st) + (v >> 1), kRsv << ((v & 1) * 16),
                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  };

  // front end: the chunk whose states are read next (its source, positions and
  // first ids), and the end of the chunk after it
  int32_t chunk = 0;
  int32_t fx = lane * stride;
  int32_t fb = 0, fe = 0;
  uint32_t pe = 0;  // as loaded: the offset's low 32 bits
  ids4 f{0, 0, 0, 0};
  uint32_t fw = 0;
  bool pending = false;
  uint32_t q_head = 0, q_tail = 0;
  if (fx < n) {
    fb = (int32_t)((int64_t)off[fx] - base);
    fe = (int32_t)((int64_t)off[fx + 1] - base);
    if (fb < fe && fb <= m4) f = *reinterpret_cast<GIds>(nbr + fb);
  }
  if (stride > 1 && fx + 1 < n) pe = (uint32_t)off[fx + 2];

  // The lanes in each phase (see sweep.h): ids requested, states requested, u
  // or v requested, waiting for u, waiting for v (with u held, or given back).
  // Lanes in none of them, nor paused for an assist, are idle.
  uint64_t p_ids = 0, p_sts = 0, p_res = 0, p_mat = 0, p_chk = 0, p_mw = 0, p_vw = 0, p_asst = 0;
  int64_t trips = 0;
  int32_t x = 0, u = 0, v = 0, i = 0, e = 0, steps = 0;
  int32_t t = 0;            // the vertex last asked for: u or v
  ids4 w{0, 0, 0, 0};       // the ids being examined
  ids4 c{0, 0, 0, 0};       // the ids at i, loaded ahead (if i <= m4)
  ids4 h{0, 0, 0, 0};       // the first ids of a source handed out on the last trip,
  uint64_t fresh = 0;       // to these lanes
  // bits of w's ids: worth a state read; not reached by a state read yet; read
  // by the current state read; seen free and not tried yet
  uint32_t cand = 0, todo = 0, rd = 0, live = 0;
  uint32_t s0 = 0, s1 = 0, s2 = 0, s3 = 0;  // their entries
  uint64_t first = 0;                       // lanes that have read no state of their source yet
  bool cut = false;                         // the list is ordered upper neighbours first
  uint32_t mat_w = 0, res_w = 0, chk_u = 0, chk_v = 0;
  // wavefront assist: its stage, where it reads ahead, the candidates found and
  // the ids below the source among them, and whether the source is matched
  int asst = 0;
  int32_t ai = 0, ae = 0, ax = 0;
  uint64_t a_cand = 0, a_low = 0, a_dead = 0;

#pragma unroll 1
  while (true) {
    // ---------------- consume the results of last trip's operations
    const uint64_t p_act = p_mat | p_res;
    const uint32_t sw = ((in(p_mat) ? mat_w : res_w) >> ((t & 1) * 16)) & 0xffffu;
    const uint64_t k_free = __ballot(sw == 0);
    const uint64_t k_dead = p_act & __ballot((sw & kMch) != 0);
    const uint64_t k_rsvd = p_act & ~k_free & ~k_dead;
    const uint64_t k_won = p_mat & k_free;
    const uint64_t k_held = p_res & k_free;
    uint64_t adv = k_dead & __ballot(t != x) | p_sts;  // these take their next candidate
    const uint64_t k_back = p_mat & (k_dead | (k_rsvd & give_back));
    if (in(k_won)) {
      st[u] = (uint16_t)(kMch | kRsv | (uint32_t)v);
      st[v] = (uint16_t)(kMch | kRsv | (uint32_t)u);
    }
    if (in(k_back)) st[u] = 0;
    if (in(p_sts))
      live = rd & ~((s0 >> 15) | ((s1 >> 14) & 2u) | ((s2 >> 13) & 4u) | ((s3 >> 12) & 8u));
    uint64_t n_sts = 0, n_ids = 0, n_res = 0, n_mat = k_held, more = 0;
    {
      if (in(p_ids & ~fresh)) w = c;
      if (in(fresh)) w = h;
      if (in(p_ids)) {
        if (i > m4) {  // the last list's last ids
          w.x = nbr[i];
          w.y = i + 1 < m ? nbr[i + 1] : 0;
          w.z = i + 2 < m ? nbr[i + 2] : 0;
          w.w = i + 3 < m ? nbr[i + 3] : 0;
        }
        const int32_t rem = e - i;
        const int32_t nids = rem < W ? rem : W;
        i += nids;
        steps += nids;
        todo = (1u << nids) - 1;
        uint32_t k;
        if (UPPER) {
          k = ((uint32_t)(x - w.x) >> 31) | ((uint32_t)(x - w.y) >> 31 << 1) |
              ((uint32_t)(x - w.z) >> 31 << 2) | ((uint32_t)(x - w.w) >> 31 << 3);
          if (a.lower_stop > 0) {
            const uint32_t low = ((uint32_t)(w.x - x) >> 31) | ((uint32_t)(w.y - x) >> 31 << 1) |
                                 ((uint32_t)(w.z - x) >> 31 << 2) | ((uint32_t)(w.w - x) >> 31 << 3);
            if (cut && (low & todo)) e = i;  // the rest of the list is below x
          }
        } else {
          k = (w.x != x ? 1u : 0u) | (w.y != x ? 2u : 0u) | (w.z != x ? 4u : 0u) | (w.w != x ? 8u : 0u);
        }
        cand = k & todo;
      }
      more = p_ids & __ballot(i < e);
      n_sts = UPPER ? p_ids & __ballot(cand != 0) : p_ids;
      n_ids = more & ~n_sts;
    }

    uint64_t n_chk = p_res & k_rsvd;
    uint64_t n_mw = p_mat & k_rsvd & ~give_back;
    uint64_t n_vw = p_mat & k_rsvd & give_back;
    if (__builtin_expect((p_chk | p_mw | p_vw) != 0, 0)) {
      const uint64_t vdead = __ballot((chk_v & kMch) != 0), vfree = __ballot(chk_v == 0);
      const uint64_t udead = __ballot((chk_u & kMch) != 0), ufree = __ballot(chk_u == 0);
      const uint64_t vx = __ballot(v == x), ux = __ballot(u == x);
      const uint64_t c_ud = p_chk & ~vdead & udead;
      const uint64_t c_free = p_chk & ~vdead & ufree;
      const uint64_t waits = p_chk | p_mw | p_vw;
      adv |= (waits & vdead & ~vx) | (c_ud & ~ux);
      n_res |= c_free | (p_vw & vfree);
      n_mat |= p_mw & vfree;
      n_chk |= p_chk & ~vdead & ~udead & ~ufree;
      n_mw |= p_mw & ~vdead & ~vfree;
      n_vw |= p_vw & ~vdead & ~vfree;
      if (in(p_mw & vdead)) st[u] = 0;
    }
    {
      const uint64_t k_live = adv & __ballot(live != 0);
      const uint64_t k_todo = adv & ~k_live & __ballot(todo != 0);
      n_ids |= adv & ~k_live & ~k_todo & __ballot(i < e);
      n_sts |= k_todo;
      n_res |= k_live;
      if (in(k_live)) {
        const int32_t l0 = (int32_t)(live << 31) >> 31, l1 = (int32_t)(live << 30) >> 31,
                      l2 = (int32_t)(live << 29) >> 31;
        int32_t y = (w.z & l2) | (w.w & ~l2);
        y = (w.y & l1) | (y & ~l1);
        y = (w.x & l0) | (y & ~l0);
        live &= live - 1;
        u = x < y ? x : y;
        v = x < y ? y : x;
      }
    }
    p_ids = n_ids;
    p_sts = n_sts;
    p_res = n_res;
    p_mat = n_mat;
    p_chk = n_chk;
    p_mw = n_mw;
    p_vw = n_vw;
    lds_order();

    // ---------------- front end: queue the chunk whose states were read
    if (pending) {
      const uint64_t need = __ballot(fx < n) & __ballot(fb != fe) & __ballot(!(fw & kMch));
      if (in(need)) {
        const uint32_t slot = (q_tail + lanes_below(need)) & (kQueue - 1);
        q.b[slot] = fb;
        q.e[slot] = fe;
        q.ids[slot] = f;
        q.x[slot] = (uint16_t)fx;
      }
      q_tail += (uint32_t)__popcll(need);
      pending = false;
      // the next chunk: its first ids, and the end of the one after it
      ++fx;
      fb = fe;
      fe = (int32_t)(pe - (uint32_t)base);
      if (chunk < stride) {
        if (in(__ballot(fx < n) & __ballot(fb < fe) & __ballot(fb <= m4)))
          f = *reinterpret_cast<GIds>(nbr + fb);
        if (chunk + 1 < stride && fx + 1 < n) pe = (uint32_t)off[fx + 2];
      }
      lds_order();
    }

    // the ids after those taken above, needed two trips from now or later (one,
    // if none of them was worth a state read)
    if (in(more & __ballot(i <= m4))) c = *reinterpret_cast<GIds>(nbr + i);

    // ---------------- wavefront assist: consume
    if (__builtin_expect(asst == 2, 0)) {
      if (in(p_asst)) {
        if (cut && a_low) e = ai + (int32_t)__builtin_ctzll(a_low);
        i = a_cand ? ai + (int32_t)__builtin_ctzll(a_cand) : (ae - ai > 64 ? ai + 64 : ae);
        steps = 0;
        if (i < e && i <= m4) c = *reinterpret_cast<GIds>(nbr + i);
      }
      // a source matched by another lane meanwhile is done
      if (!a_dead) p_ids |= p_asst & __ballot(i < e);
      p_asst = 0;
      asst = 0;
    }

    // the lanes whose scans have become long (never one handed a source now)
    uint64_t longs = 0;
    if (a.assist_after > 0) longs = p_ids & __ballot(steps >= a.assist_after) & __ballot(e - i > 2 * W);

    // ---------------- hand queued sources to idle lanes
    fresh = 0;
    const uint64_t idle = ~(p_ids | p_sts | p_res | p_mat | p_chk | p_mw | p_vw | p_asst);
    const uint32_t avail = q_tail - q_head;
    if (avail) {
      const uint32_t r = lanes_below(idle);
      const uint64_t take = idle & __ballot(r < avail);
      if (in(take)) {
        const uint32_t slot = (q_head + r) & (kQueue - 1);
        i = __hip_atomic_load(q.b + slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
        e = __hip_atomic_load(q.e + slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
        h = q.ids[slot];
        x = q.x[slot];
        steps = 0;
        if (UPPER && a.lower_stop > 0) cut = e - i <= a.lower_stop;
      }
      fresh = take;
      first |= take;
      p_ids |= take;
      q_head += (uint32_t)__popcll(take);
      lds_order();
    } else if (chunk >= stride && !~idle) {
      break;  // every source handed out and done (no chunk is pending here)
    }
    if (++trips > cap) {
      if (lane == 0) atomicOr(a.err, 1u);
      break;
    }

    // ---------------- issue one operation per lane. The front end and the
    // assist below only look at matched bits, which change above alone, so
    // their work may come after it and under its latency; the sources handed
    // out above are first looked at on the next trip
    t = in(p_res) ? u : v;
    if (__builtin_expect((p_mw | p_vw) != 0, 0)) {
      if (in(p_mw | p_vw)) chk_v = st[v];
      lds_order();
    }
    if (in(p_mat)) mat_w = reserve(t);
    lds_order();
    if (__builtin_expect(p_chk != 0, 0)) {
      if (in(p_chk)) {
        chk_u = st[u];
        chk_v = st[v];
      }
      lds_order();
    }
    if (in(p_res)) res_w = reserve(t);
    lds_order();
    if (in(p_sts)) {
      rd = cand & todo;
      const uint32_t t0 = todo;
      todo = 0;
      if (in(p_sts & (one_all | (first & one_first)))) {
        rd &= 0u - rd;  // the first candidate
        todo = rd ? t0 & ~(rd | (rd - 1)) : 0u;  // the positions behind it
      }
      s0 = st[w.x];
      s1 = st[w.y];
      s2 = st[w.z];
      s3 = st[w.w];
    }
    first &= ~p_sts;
    lds_order();

    // ---------------- front end: read the states of the next chunk's sources
    if (chunk < stride && q_tail - q_head < 64) {
      ++chunk;
      if (fx < n) fw = st[fx];
      pending = true;
    }

    // ---------------- wavefront assist: issue
    if (__builtin_expect(asst == 1, 0)) {
      const int32_t id = (int32_t)(int16_t)q.ahead[lane];
      const bool have = id >= 0;
      a_cand = __ballot(have && id != ax && (!UPPER || id > ax) && !(st[have ? id : 0] & kMch));
      a_low = a.lower_stop > 0 ? __ballot(have && id < ax) : 0;
      a_dead = __ballot((st[ax] & kMch) != 0);
      asst = 2;
    } else if (__builtin_expect(longs != 0, 0)) {
      const int al = __builtin_ctzll(longs);
      ai = __builtin_amdgcn_readlane(i, al);
      ae = __builtin_amdgcn_readlane(e, al);
      ax = __builtin_amdgcn_readlane(x, al);
      p_asst = longs & (0 - longs);
      p_ids &= ~p_asst;
      q.ahead[lane] = ai + lane < ae ? (uint16_t)nbr[ai + lane] : (uint16_t)0xffff;
      asst = 1;
      lds_order();
    }

    lds_order();
  }
}

// Sweeps the sources 0 .. n-1 of one graph with this wavefront, using lds
// (at least whole_lds_words(n) words of LDS) and the ring q. mate: the
// graph's output (n entries, device memory), written for every vertex at the
// end. The instrumented build runs sweep_block itself on these states: the
// counters it reports are those of the same schedule.
template <typename OffT, bool STATS>
__device__ __forceinline__ void sweep_whole_lds(SweepParams p, const OffT* __restrict__ off,
                                                const int32_t* __restrict__ nbr, int64_t n,
                                                int32_t* mate, uint32_t* lds, QSlot* q,
                                                Counters<STATS>& cnt) {
  const int lane = (int)(threadIdx.x & 63);
  // the graph is in device memory: global loads, which the waits for LDS
  // results do not include (flat loads would be counted with them)
  using GOff = const __attribute__((address_space(1))) OffT*;
  using GNbr = const __attribute__((address_space(1))) int32_t*;
  const int64_t m = (int64_t)off[n] - (int64_t)off[0];
  if (!STATS && m >= 0 && m <= kWholeEntries) {
    lds_u16* st = reinterpret_cast<lds_u16*>(lds);
    for (int64_t i = lane; i < whole_entry_words(n) / 4; i += 64)
      reinterpret_cast<uint4*>(lds)[i] = make_uint4(0u, 0u, 0u, 0u);  // every vertex ACC
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    WholeQueue& wq = *reinterpret_cast<WholeQueue*>(q);
    if (p.upper_only)
      whole_loop<OffT, true>(p, (GOff)off, (GNbr)nbr, (int32_t)n, (int32_t)m, st, wq);
    else
      whole_loop<OffT, false>(p, (GOff)off, (GNbr)nbr, (int32_t)n, (int32_t)m, st, wq);
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    // eight entries per lane and step: their reads are in flight together
    for (int32_t v0 = lane; v0 < (int32_t)n; v0 += 512) {
      uint32_t s[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) s[k] = v0 + 64 * k < (int32_t)n ? st[v0 + 64 * k] : 0u;
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (v0 + 64 * k < (int32_t)n)
          mate[v0 + 64 * k] = (s[k] & 0x8000u) ? (int32_t)(s[k] & 0x3fffu) : -1;
    }
    return;
  }
  const int64_t words = whole_state_words(n);
  for (int64_t i = lane; i < words; i += 64) lds[i] = 0u;  // every vertex ACC
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
  p.wave_vertices = (n + 63) / 64 * 64;
  p.disperse = 1;  // lanes stride apart (see the whole-graph case of mm_run)
  p.hub_degree = 0;
  p.chunks = nullptr;
  LayoutLds lay;
  lay.w = lds;
  lay.mate = nullptr;
  lay.hint = Hint{nullptr, 0};
  lay.mate16 = reinterpret_cast<int16_t*>(lds + words);
  sweep_block<OffT, LayoutLds, false, false, STATS, false, GOff, GNbr>(p, (GOff)off, (GNbr)nbr, lay, 0, n,
                                                                q, nullptr, cnt);
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
  // every lane is done, so no vertex is still reserved: a state is ACC or MCHD
  for (int64_t v = lane; v < n; v += 64)
    mate[v] = LayoutLds::matched(lds[v >> 4], v) ? (int32_t)lay.mate16[v] : -1;
}

}  // namespace mmk
