// Solve-phase setup: the Gauss-Seidel colouring of each A_l, the
// colour-sorted solve layout (SELL-64 matrix, SoA prolongation, restriction
// rows), and the dense factorisation of the coarsest operator (Alg. 2 solves
// the coarsest level directly).
#include <utility>
#include <algorithm>
#include <cstring>

#include "gmg_internal.hpp"

namespace gmg {

namespace {

// ------------------------------------------------------------------ colouring
// Greedy first-fit colouring in hashed key order, run as Jones-Plassmann
// rounds: a row is coloured once all its lower-key neighbours are, with the
// smallest colour none of them uses.  Decisions are final, so colours are
// written in place.
struct ColorKey {
  uint64_t base;
  __device__ uint64_t operator()(int32_t v) const { return mix64(base ^ (uint64_t)v); }
};

constexpr int kColorChunk = 16;

// On levels of up to kColorListLevel rows the first visit of v also records
// the lower-key neighbours not yet coloured, in list[v * kColorList ..] with
// their number in cnt[v], and the colours of those already coloured as a bit
// mask (cnt[v] = kColorList + 1: too many neighbours to list, or a colour of
// 64 or more; later visits read the row again).  Colours are final once
// written, so a later visit reads only the listed neighbours' colours and
// takes the same decision as a visit that reads the whole row.
constexpr int kColorList = 32;
constexpr int64_t kColorListLevel = 262144;

struct ColorLists {
  int32_t* list = nullptr;   // null: no lists, every visit reads the row
  uint64_t* mask = nullptr;
  uint8_t* cnt = nullptr;
};

__device__ inline int32_t first_fit_above(const int32_t* rp, const int32_t* col, const ColorKey& key,
                                          const int32_t* color, int32_t v, uint64_t kv) {
  for (int32_t c = 64;; ++c) {                  // rare: every colour below 64 is taken
    bool used = false;
    for (int32_t e = rp[v]; e < rp[v + 1] && !used; ++e) {
      int32_t u = col[e];
      if (u == v) continue;
      uint64_t ku = key(u);
      if ((ku < kv || (ku == kv && u < v)) && color[u] == c) used = true;
    }
    if (!used) return c;
  }
}

// Returns 0 if v must wait for a lower-key neighbour, else colours v and
// returns its colour + 1.  The row is read kColorChunk entries at a time with
// every column and neighbour-colour load in flight together (positions past
// the row's end re-read its last entry; every row holds its diagonal).  With
// Record, a waiting row also writes its lists.
template <bool Record>
__device__ inline int32_t color_attempt(const int32_t* rp, const int32_t* col, const ColorKey& key,
                                        int32_t* color, int32_t v, const ColorLists& L) {
  const uint64_t kv = key(v);
  uint64_t mask = 0;
  bool high = false, wait = false;
  int32_t nrec = 0;
  const int32_t b = rp[v], e = rp[v + 1];
  for (int32_t e0 = b; e0 < e; e0 += kColorChunk) {
    int32_t u[kColorChunk], cu[kColorChunk];
#pragma unroll
    for (int k = 0; k < kColorChunk; ++k) u[k] = col[min(e0 + k, e - 1)];
#pragma unroll
    for (int k = 0; k < kColorChunk; ++k) cu[k] = __atomic_load_n(&color[u[k]], __ATOMIC_RELAXED);
#pragma unroll
    for (int k = 0; k < kColorChunk; ++k) {
      if (e0 + k >= e || u[k] == v) continue;
      const uint64_t ku = key(u[k]);
      if (!(ku < kv || (ku == kv && u[k] < v))) continue;
      if (cu[k] < 0) {
        wait = true;
        if constexpr (Record) {
          if (nrec < kColorList) L.list[(int64_t)v * kColorList + nrec] = u[k];
          ++nrec;
        }
      } else if (cu[k] < 64) {
        mask |= 1ull << cu[k];
      } else {
        high = true;
      }
    }
  }
  if (wait) {
    if constexpr (Record) {
      L.mask[v] = mask;
      L.cnt[v] = (uint8_t)(nrec <= kColorList && !high ? nrec : kColorList + 1);
    }
    return 0;
  }
  int32_t c = (~mask) ? __builtin_ctzll(~mask) : 64;
  if (c == 64 && high) c = first_fit_above(rp, col, key, color, v, kv);
  color[v] = c;
  return c + 1;
}

// A later visit of a row with lists: the colours of the listed neighbours.
__device__ inline int32_t color_again(const int32_t* rp, const int32_t* col, const ColorKey& key,
                                      int32_t* color, int32_t v, const ColorLists& L) {
  const int32_t n = L.cnt[v];
  if (n > kColorList) return color_attempt<false>(rp, col, key, color, v, L);
  uint64_t mask = L.mask[v];
  bool high = false, wait = false;
  const int32_t* lp = L.list + (int64_t)v * kColorList;
  for (int32_t e0 = 0; e0 < n; e0 += kColorChunk) {
    int32_t u[kColorChunk], cu[kColorChunk];
#pragma unroll
    for (int k = 0; k < kColorChunk; ++k) u[k] = lp[min(e0 + k, n - 1)];
#pragma unroll
    for (int k = 0; k < kColorChunk; ++k) cu[k] = __atomic_load_n(&color[u[k]], __ATOMIC_RELAXED);
#pragma unroll
    for (int k = 0; k < kColorChunk; ++k) {
      if (e0 + k >= n) continue;
      if (cu[k] < 0) wait = true;
      else if (cu[k] < 64) mask |= 1ull << cu[k];
      else high = true;
    }
  }
  if (wait) return 0;
  int32_t c = (~mask) ? __builtin_ctzll(~mask) : 64;
  if (c == 64 && high) c = first_fit_above(rp, col, key, color, v, key(v));
  color[v] = c;
  return c + 1;
}

// Any visit: the first (round 0 over every row) records the lists.
__device__ inline int32_t color_visit(const int32_t* rp, const int32_t* col, const ColorKey& key, int32_t* color,
                                      int32_t v, const ColorLists& L, bool first) {
  if (!L.list) return color_attempt<false>(rp, col, key, color, v, L);
  if (first) return color_attempt<true>(rp, col, key, color, v, L);
  return color_again(rp, col, key, color, v, L);
}

// One Jones-Plassmann round; round 0 visits every row, later rounds the
// worklist of rows still waiting after the previous round.
__global__ void __launch_bounds__(kBlock) k_color_round(const int32_t* rp, const int32_t* col, int64_t n,
                                                        ColorKey key, int32_t* color, const int32_t* wl_in,
                                                        int32_t* wl_out, int32_t* rounds, int k, ColorLists L) {
  const int64_t count = k == 0 ? n : rounds[k - 1];
  for (int64_t base = (int64_t)blockIdx.x * kBlock; base < count; base += (int64_t)gridDim.x * kBlock) {
    const int64_t i = base + threadIdx.x;
    const bool act = i < count;
    const int32_t v = act ? (k == 0 ? (int32_t)i : wl_in[i]) : 0;
    int32_t got = 0;
    if (act) got = color_visit(rp, col, key, color, v, L, k == 0);
    block_append(act && got == 0, v, wl_out, &rounds[k]);
  }
}

// One class of an iterated-greedy pass: every vertex v with old[v] == c takes
// the smallest colour not used by a neighbour's new colour (neu[u] >= 0: the
// classes above c, recoloured by earlier launches).  Vertices of one class are
// not adjacent, so they are recoloured in parallel.
__global__ void __launch_bounds__(kBlock) k_ig_class(const int32_t* rp, const int32_t* col, int64_t n,
                                                     const int32_t* old, int32_t* neu, int32_t c) {
  for (int64_t v = (int64_t)xcd_block() * kBlock + threadIdx.x; v < n; v += (int64_t)gridDim.x * kBlock) {
    if (old[v] != c) continue;
    const int32_t b = rp[v], e = rp[v + 1];
    uint64_t mask = 0;
    bool high = false;
    for (int32_t e0 = b; e0 < e; e0 += kColorChunk) {
      int32_t u[kColorChunk], cu[kColorChunk];
#pragma unroll
      for (int k = 0; k < kColorChunk; ++k) u[k] = col[min(e0 + k, e - 1)];
#pragma unroll
      for (int k = 0; k < kColorChunk; ++k) cu[k] = neu[u[k]];
#pragma unroll
      for (int k = 0; k < kColorChunk; ++k) {
        if (e0 + k >= e || u[k] == v || cu[k] < 0) continue;
        if (cu[k] < 64) mask |= 1ull << cu[k];
        else high = true;
      }
    }
    int32_t k = (~mask) ? __builtin_ctzll(~mask) : 64;
    if (k == 64 && high) {
      for (;; ++k) {                            // rare: every colour below 64 is taken
        bool used = false;
        for (int32_t t = b; t < e && !used; ++t) used = col[t] != v && neu[col[t]] == k;
        if (!used) break;
      }
    }
    neu[v] = k;
  }
}

// A whole small level in one workgroup of kDrainItems threads, its row
// offsets, 16-bit columns and colours in LDS: the Jones-Plassmann rounds (the
// same first-fit decisions in key order as the multi-launch rounds), then
// `passes` iterated-greedy passes (the classes of the first colouring from the
// highest down, as k_ig_class).  Each row is first partitioned in place, its
// lower-key neighbours first, so that the rounds compute no keys; the rounds
// visit a worklist of the rows still waiting, and each pass lists the rows of
// every class.  What bounds it is the chain of a round or class, a hundred rows
// and dependent LDS reads: 16 lanes take a row, an entry each, and join their
// masks.  (With one thread a row a round took 7,900 cycles and a class 5,000:
// 1,463 rows 202 us, now 119; 2,374 rows 306 us, now 187.  Rows of more than 64 entries
// are partitioned by one of their lanes: 400 rows of 106 entries 2,800 us, now 510, and
// 130 points all coupled among 700 18.4 ms, now 17.0.)
// Writes the colours and their count.
constexpr int kSmallColorRows = 4096;
constexpr int kSmallColorPer = kSmallColorRows / kDrainItems;
constexpr int kSmallColorMax = 256;               // classes a pass can list
constexpr int64_t kSmallColorLds = 150 * 1024;
inline int64_t small_color_lds(int64_t n, int64_t nnz) {
  auto up = [](int64_t b) { return (b + 15) & ~(int64_t)15; };
  return up((n + 1) * 4) + up(nnz * 2) + 5 * up(n * 2) + up(n * 4);
}

// Smallest colour from the neighbours' mask, or, when every colour below 64
// is taken, the smallest colour no entry of scol[lo, hi) other than v has.
__device__ inline int32_t small_first_fit(const uint16_t* scol, int32_t lo, int32_t hi, const int16_t* c,
                                          int32_t v, uint64_t mask, bool high) {
  int32_t k = (~mask) ? __builtin_ctzll(~mask) : 64;
  if (k < 64 || !high) return k;
  for (;; ++k) {                                // rare: every colour below 64 is taken
    bool used = false;
    for (int32_t e = lo; e < hi && !used; ++e) used = scol[e] != v && c[scol[e]] == k;
    if (!used) return k;
  }
}

// The colours taken around a row, by the 16 lanes that share it.
struct TakenColors {
  uint32_t lo = 0, hi = 0, above = 0;            // below 32, below 64, any beyond
  __device__ void add(int32_t c, bool on) {
    const uint32_t bit = on ? 1u << (c & 31) : 0u;
    lo |= c < 32 ? bit : 0u;
    hi |= c >= 32 && c < 64 ? bit : 0u;
    above |= c >= 64 ? bit : 0u;
  }
  __device__ static uint32_t join16(uint32_t v) {   // OR over a row of 16 lanes
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xF, 0xF, false);   // rotated by 8, 4, 2, 1
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x124, 0xF, 0xF, false);
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x122, 0xF, 0xF, false);
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x121, 0xF, 0xF, false);
    return v;
  }
  __device__ void join() {
    lo = join16(lo);
    if (__ballot((hi | above) != 0)) {
      hi = join16(hi);
      above = join16(above);
    }
  }
  __device__ uint64_t mask() const { return (uint64_t)hi << 32 | lo; }
};
constexpr int kSmallLanes = 16, kSmallGroups = kDrainItems / kSmallLanes;
constexpr int kSmallRow = 4 * kSmallLanes;       // entries of a row that its lanes partition together

__global__ void __launch_bounds__(kDrainItems) k_color_small(const int32_t* rp, const int32_t* col, int32_t n,
                                                             ColorKey key, int32_t passes, int32_t* color,
                                                             int32_t* ncolors, int32_t* flags) {
  extern __shared__ int32_t lds_small[];
  auto up = [](int64_t b) { return (int32_t)((b + 15) & ~(int64_t)15); };
  char* base = reinterpret_cast<char*>(lds_small);
  int32_t* srp = reinterpret_cast<int32_t*>(base);
  const int32_t nnz = rp[n];
  uint16_t* scol = reinterpret_cast<uint16_t*>(base + up((int64_t)(n + 1) * 4));
  const int32_t na = up((int64_t)n * 2) / 2;       // int16 elements per n-array
  int16_t* ca = reinterpret_cast<int16_t*>(base + up((int64_t)(n + 1) * 4) + up((int64_t)nnz * 2));
  int16_t* cb = ca + na;
  int16_t* lowc = cb + na;                       // lower-key neighbours of each row
  int16_t* wa = lowc + na;                       // worklists / class lists
  int16_t* wb = wa + na;
  int32_t* waitc = reinterpret_cast<int32_t*>(wb + na);   // uncoloured lower-key neighbours of each row
  __shared__ int32_t s_cnt[3];
  __shared__ int32_t s_cls[kSmallColorMax + 1];
  const int tid = (int)threadIdx.x;
  for (int32_t i = tid; i <= n; i += kDrainItems) srp[i] = rp[i];
  for (int32_t i = tid; i < n; i += kDrainItems) ca[i] = -1;
  if (tid < 3) s_cnt[tid] = 0;
  // columns: 16 loads in flight per thread before their stores
  for (int32_t e0 = 0; e0 < nnz; e0 += 16 * kDrainItems) {
    int32_t cv[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) cv[u] = col[min(e0 + u * kDrainItems + tid, nnz - 1)];
#pragma unroll
    for (int u = 0; u < 16; ++u)
      if (e0 + u * kDrainItems + tid < nnz) scol[e0 + u * kDrainItems + tid] = (uint16_t)cv[u];
  }
  uint64_t* keys = reinterpret_cast<uint64_t*>(wa);   // until the worklists and counts take their place
  for (int32_t i = tid; i < n; i += kDrainItems) keys[i] = key(i);
  __syncthreads();
  const int grp = tid / kSmallLanes, t16 = tid % kSmallLanes;
  // the rows' lower-key neighbours first
  for (int32_t v = grp; v < n; v += kSmallGroups) {
    const uint64_t kv = keys[v];
    const int32_t b = srp[v], len = srp[v + 1] - b;
    auto lower = [&](int32_t u) {
      const uint64_t ku = keys[u];
      return u != v && (ku < kv || (ku == kv && u < v));
    };
    if (len <= kSmallRow) {
      int32_t u[4], at = 0;
      uint32_t low[4];                             // the lanes whose entry is lower
      const int shift = (tid & (kWave - 1)) & ~(kSmallLanes - 1);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int32_t t = t16 + k * kSmallLanes;
        u[k] = t < len ? (int32_t)scol[b + t] : -1;
        low[k] = (uint32_t)(__ballot(u[k] >= 0 && lower(u[k])) >> shift) & 0xFFFFu;
        at += __popc(low[k]);
      }
      if (t16 == 0) lowc[v] = (int16_t)at;
      int32_t nl = 0, nh = at;                     // placed so far: lower entries, others
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t below = (1u << t16) - 1u, mine = low[k] >> t16 & 1u;
        const int32_t dst = mine ? nl + __popc(low[k] & below) : nh + t16 - __popc(low[k] & below);
        if (u[k] >= 0) scol[b + dst] = (uint16_t)u[k];
        nl += __popc(low[k]);
        nh += kSmallLanes - __popc(low[k]);
      }
    } else if (t16 == 0) {
      int32_t w = b;
      for (int32_t t = b; t < b + len; ++t) {
        const int32_t u = scol[t];
        if (lower(u)) {
          scol[t] = scol[w];
          scol[w] = (uint16_t)u;
          ++w;
        }
      }
      lowc[v] = (int16_t)(w - b);
    }
  }
  __syncthreads();
  // Rounds in dependency order: a row is ready once all its lower-key
  // neighbours are coloured (its count of uncoloured ones, held in wait[],
  // reaches zero); round r colours the rows that became ready in round r - 1
  // (round 0: the rows without lower-key neighbours) and counts down their
  // higher-key neighbours, appending those that become ready, counted in
  // s_cnt[r % 3] (reset at the start of round r - 1, after every thread read
  // the count it held before).  Each coupling is visited twice in all.
  const int lane = tid & (kWave - 1);
  int32_t count = 0;
  if (tid == 0) s_cnt[0] = 0;
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kSmallColorPer; ++q) {
    const int32_t v = tid + q * kDrainItems;
    const bool ready = v < n && lowc[v] == 0;
    if (v < n) waitc[v] = lowc[v];
    const unsigned long long m = __ballot(ready);
    if (m) {
      int32_t o = 0;
      if (lane == 0) o = atomicAdd(&s_cnt[0], (int32_t)__popcll(m));
      o = __shfl(o, 0, kWave);
      if (ready) wb[o + __popcll(m & ((1ull << lane) - 1ull))] = (int16_t)v;
    }
  }
  __syncthreads();
  count = s_cnt[0];
  int32_t coloured = 0;
  bool done = count == 0;
  for (int round = 0; round < kMaxRounds && !done; ++round) {
    const int16_t* src = (round & 1) ? wa : wb;
    int16_t* dst = (round & 1) ? wb : wa;
    if (tid == 0) s_cnt[(round + 2) % 3] = 0;
    for (int32_t i = grp; i < count; i += kSmallGroups) {
      const int32_t v = src[i];
      const int32_t b = srp[v], l = b + lowc[v];
      TakenColors taken;                             // by the lower-key neighbours, all coloured
      for (int32_t t = b + t16; t < l; t += kSmallLanes) taken.add(ca[scol[t]], true);
      taken.join();
      if (t16 == 0) ca[v] = (int16_t)small_first_fit(scol, b, l, ca, v, taken.mask(), taken.above != 0);
    }
    __syncthreads();                              // the round's colours are written
    // count down the higher-key neighbours of the round's rows
    for (int32_t i = grp; i < count; i += kSmallGroups) {
      const int32_t v = src[i];
      const int32_t e = srp[v + 1];
      for (int32_t t = srp[v] + lowc[v] + t16; t < e; t += kSmallLanes) {
        const int32_t u = scol[t];
        if (u != v && atomicSub(&waitc[u], 1) == 1) dst[atomicAdd(&s_cnt[(round + 1) % 3], 1)] = (int16_t)u;
      }
    }
    coloured += count;
    __syncthreads();
    count = s_cnt[(round + 1) % 3];
    done = count == 0;
  }
  done = coloured == n;
  if (!done) {
    if (tid == 0) atomicOr(flags, F_TIMEOUT);
    return;
  }
  // the count of colours
  if (tid == 0) s_cnt[0] = 0;
  __syncthreads();
  {
    int32_t m = 0;
    for (int32_t v = tid; v < n; v += kDrainItems) m = max(m, (int32_t)ca[v] + 1);
    atomicMax(&s_cnt[0], m);
  }
  __syncthreads();
  const int32_t nc0 = s_cnt[0];
  if (nc0 > kSmallColorMax) {
    if (tid == 0) atomicOr(flags, F_OVERFLOW);
    return;
  }
  int16_t* cur = ca;
  int16_t* nxt = cb;
  if (nc0 > 1) {
    for (int p = 0; p < passes; ++p) {
      // the rows of every class of cur, listed in wa (any order within a class)
      for (int32_t c = tid; c <= nc0; c += kDrainItems) s_cls[c] = 0;
      __syncthreads();
      for (int32_t v = tid; v < n; v += kDrainItems) {
        atomicAdd(&s_cls[cur[v] + 1], 1);
        nxt[v] = -1;
      }
      __syncthreads();
      if (tid == 0)
        for (int32_t c = 1; c <= nc0; ++c) s_cls[c] += s_cls[c - 1];
      __syncthreads();
      for (int32_t v = tid; v < n; v += kDrainItems) wa[atomicAdd(&s_cls[cur[v]], 1)] = (int16_t)v;
      __syncthreads();
      // after the placement s_cls[c] is the end of class c (its start: s_cls[c - 1], or 0)
      for (int32_t c = nc0 - 1; c >= 0; --c) {
        const int32_t lo = c > 0 ? s_cls[c - 1] : 0, hi = s_cls[c];
        for (int32_t i = lo + grp; i < hi; i += kSmallGroups) {
          const int32_t v = wa[i];
          const int32_t b = srp[v], e = srp[v + 1];
          TakenColors taken;
          for (int32_t t = b + t16; t < e; t += kSmallLanes) {
            const int32_t u = scol[t], c = nxt[u];
            taken.add(c, u != v && c >= 0);
          }
          taken.join();
          if (t16 == 0) nxt[v] = (int16_t)small_first_fit(scol, b, e, nxt, v, taken.mask(), taken.above != 0);
        }
        __syncthreads();
      }
      int16_t* t = cur;
      cur = nxt;
      nxt = t;
    }
  }
  if (tid == 0) s_cnt[0] = 0;
  __syncthreads();
  int32_t m = 0;
  for (int32_t v = tid; v < n; v += kDrainItems) {
    color[v] = cur[v];
    m = max(m, (int32_t)cur[v] + 1);
  }
  atomicMax(&s_cnt[0], m);
  __syncthreads();
  if (tid == 0) *ncolors = s_cnt[0];
}

// The remaining Jones-Plassmann rounds in one workgroup, once at most
// kDrainItems rows wait: count_in rows in wl_in (or, if wl_in is null, all
// rows 0 .. n - 1).
__global__ void __launch_bounds__(kDrainItems) k_color_drain(const int32_t* rp, const int32_t* col, int64_t n,
                                                             ColorKey key, int32_t* color, const int32_t* wl_in,
                                                             const int32_t* count_in, ColorLists L, int32_t* flags) {
  __shared__ int32_t buf[2][kDrainItems];
  __shared__ int32_t c;
  int32_t count = wl_in ? *count_in : (int32_t)n;
  int cur = 0;
  for (int round = 0; round < kMaxRounds; ++round) {
    if (threadIdx.x == 0) c = 0;
    __syncthreads();
    if ((int32_t)threadIdx.x < count) {
      const int32_t v = round == 0 ? (wl_in ? wl_in[threadIdx.x] : (int32_t)threadIdx.x) : buf[cur][threadIdx.x];
      if (!color_visit(rp, col, key, color, v, L, round == 0 && !wl_in)) buf[cur ^ 1][atomicAdd(&c, 1)] = v;
    }
    __syncthreads();
    count = c;
    cur ^= 1;
    __syncthreads();
    if (count == 0) return;
  }
  if (threadIdx.x == 0) atomicOr(flags, F_TIMEOUT);
}

// ------------------------------------------------------------------ stable colour partition
// hist[c * nb + b] = rows of colour c in block b; its exclusive scan gives,
// for every (colour, block), the first new index, so new indices are sorted
// by (colour, old index).
__global__ void __launch_bounds__(kBlock) k_color_hist(const int32_t* color, int64_t n, int nb, int nc,
                                                       int32_t* hist) {
  extern __shared__ int32_t cnt[];
  for (int c = threadIdx.x; c < nc; c += blockDim.x) cnt[c] = 0;
  __syncthreads();
  int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (v < n) atomicAdd(&cnt[color[v]], 1);
  __syncthreads();
  for (int c = threadIdx.x; c < nc; c += blockDim.x) hist[(int64_t)c * nb + blockIdx.x] = cnt[c];
}

// order: the points the keys belong to (null: point v has key v)
__global__ void __launch_bounds__(kBlock) k_color_place(const int32_t* color, int64_t n, int nb, const int32_t* off,
                                                        const int32_t* order, int32_t* perm, int32_t* iperm) {
  __shared__ int32_t cl[kBlock];
  int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  cl[threadIdx.x] = v < n ? color[v] : -1;
  __syncthreads();
  if (v >= n) return;
  int32_t c = cl[threadIdx.x], rank = 0;
  for (int t = 0; t < (int)threadIdx.x; ++t) rank += cl[t] == c;
  int32_t nw = off[(int64_t)c * nb + blockIdx.x] + rank;
  const int32_t p = order ? order[v] : (int32_t)v;
  perm[nw] = p;
  iperm[p] = nw;
}

// Rows whose first coupling lies within kNear of the next row's, of n - 1.
constexpr int32_t kNear = 32;
__global__ void __launch_bounds__(kBlock) k_near_rows(const int32_t* __restrict__ rp, const int32_t* __restrict__ col,
                                                      int64_t n, int32_t* near) {
  auto first = [&](int64_t i) {
    const int32_t b = rp[i], e = rp[i + 1];
    return b < e ? (col[b] != (int32_t)i || b + 1 == e ? col[b] : col[b + 1]) : (int32_t)i;
  };
  int32_t m = 0;
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i + 1 < n; i += (int64_t)gridDim.x * kBlock)
    m += abs(first(i + 1) - first(i)) <= kNear ? 1 : 0;
  m = block_reduce(m, [](int32_t a, int32_t b) { return a + b; });
  if (threadIdx.x == 0) atomicAdd(near, m);
}

// pos[j] = position of coarse point j among the rows listed block by block.
__global__ void k_block_pos(const int32_t* brows, const int32_t* perm, int64_t nc, int32_t* pos) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p < nc) pos[perm[brows[p]]] = (int32_t)p;
}

__global__ void k_gather_i32(const int32_t* in, const int32_t* idx, int64_t n, int32_t* out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = in[idx[i]];
}

__global__ void k_cluster_count(const int32_t* label, const int32_t* pos, int64_t n, int32_t* cnt, int32_t* slot) {
  const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (v < n) slot[v] = atomicAdd(&cnt[pos[max(label[v], 0)]], 1);
}

__global__ void k_cluster_place(const int32_t* label, const int32_t* pos, const int32_t* ptr, const int32_t* slot,
                                int64_t n, int32_t* order) {
  const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (v < n) order[ptr[pos[max(label[v], 0)]] + slot[v]] = (int32_t)v;
}

// cptr[c] = first new index of colour c (keys of stride classes per colour).
__global__ void k_color_ptr(const int32_t* off, int nb, int nc, int stride, int32_t* cptr) {
  int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c <= nc) cptr[c] = off[(int64_t)c * stride * nb];
}

// key = colour * kLenKeys + class, the class counting down from the widest
// rows (in 4-entry quads), so that a colour's rows come longest first.
__global__ void k_len_class(const int32_t* color, const int32_t* rp, int64_t n, int32_t* key) {
  const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= n) return;
  const int32_t quads = (rp[v + 1] - rp[v] + 3) / 4;
  key[v] = color[v] * kLenKeys + (kLenKeys - 1 - min(max(quads - 1, 0), kLenKeys - 1));
}

// ------------------------------------------------------------------ SELL-64 matrices
// Row r of the result is source row perm[r] (or r) of a CSR matrix; columns
// are renumbered through cmap (or kept); entries keep their CSR order, so
// every row sum adds its terms in the same order as the source row.
// Row lengths, slice sizes and the longest row in one pass: one thread per
// row over whole slices (a wavefront's 64 rows are one slice, so the slice
// width is a wavefront maximum); *mx = max(*mx, longest row).
__global__ void __launch_bounds__(kBlock) k_row_len_width(const int32_t* __restrict__ perm,
                                                          const int32_t* __restrict__ rp, int64_t n, int64_t ns,
                                                          int32_t* __restrict__ len, int32_t* __restrict__ wsz,
                                                          int32_t* mx) {
  const int64_t r = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  int32_t l = 0;
  if (r < n) {
    const int32_t src = perm ? perm[r] : (int32_t)r;
    l = rp[src + 1] - rp[src];
    len[r] = l;
  }
  int32_t w = l;
  for (int o = kWave / 2; o > 0; o >>= 1) w = max(w, __shfl_xor(w, o, kWave));
  const int64_t sl = r / kSlice;
  if ((threadIdx.x & (kWave - 1)) == 0 && sl < ns) wsz[sl] = w * kSlice;
  const int32_t b = block_reduce(l, [](int32_t a, int32_t c) { return a > c ? a : c; });
  if (threadIdx.x == 0 && b) atomicMax(mx, b);
}

constexpr int kFillChunk = 8;

// The loads of kFillChunk entries of the source row are issued together
// (positions past the row's end re-read its last entry and store padding).
__global__ void k_sell_fill(const int32_t* __restrict__ perm, const int32_t* __restrict__ cmap,
                            const int32_t* __restrict__ rp, const int32_t* __restrict__ col,
                            const double* __restrict__ val, int64_t n, const int32_t* __restrict__ sptr,
                            int32_t* __restrict__ scol, double* __restrict__ sval, double* __restrict__ diag) {
  int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n) return;
  int64_t s = r / kSlice, ln = r % kSlice;
  int32_t src = perm ? perm[r] : (int32_t)r;
  const int32_t b = rp[src], len = rp[src + 1] - b;
  const int32_t base = sptr[s];
  const int32_t w = (sptr[s + 1] - base) / kSlice;
  for (int32_t t0 = 0; t0 < w; t0 += kFillChunk) {
    int32_t j[kFillChunk], m[kFillChunk];
    double v[kFillChunk];
    if (len > 0) {
#pragma unroll
      for (int k = 0; k < kFillChunk; ++k) {
        const int32_t q = b + min(t0 + k, len - 1);
        j[k] = col[q];
        v[k] = val[q];
      }
#pragma unroll
      for (int k = 0; k < kFillChunk; ++k) m[k] = cmap ? cmap[j[k]] : j[k];
    }
#pragma unroll
    for (int k = 0; k < kFillChunk; ++k) {
      const int32_t t = t0 + k;
      if (t >= w) break;
      const int64_t o = base + (int64_t)t * kSlice + ln;
      if (t < len) {
        scol[o] = m[k];
        sval[o] = v[k];
        if (diag && j[k] == src) diag[r] = v[k];
      } else {
        scol[o] = 0;
        sval[o] = 0.0;
      }
    }
  }
}

// The same fill, one workgroup per slice of 64 rows, transposed through LDS:
// every source row is read contiguously (its entries across lanes), the slice
// is written column by column (entry t of the 64 rows contiguous).  pitch is
// at least the longest row of the matrix.
constexpr int kSliceFillMax = 64;

__global__ void __launch_bounds__(kBlock) k_sell_fill_slice(const int32_t* __restrict__ perm,
                                                            const int32_t* __restrict__ cmap,
                                                            const int32_t* __restrict__ rp,
                                                            const int32_t* __restrict__ col,
                                                            const double* __restrict__ val, int64_t n,
                                                            const int32_t* __restrict__ sptr,
                                                            int32_t* __restrict__ scol, double* __restrict__ sval,
                                                            double* __restrict__ diag, int pitch) {
  extern __shared__ double fill_lds[];
  double* lv = fill_lds;                                   // [kSlice][pitch]
  int32_t* lc = (int32_t*)(fill_lds + kSlice * pitch);     // [kSlice][pitch]
  __shared__ int32_t rb[kSlice], rl[kSlice], rs[kSlice];
  const int64_t s = xcd_block();
  const int64_t r0 = s * kSlice;
  const int tid = threadIdx.x;
  if (tid < kSlice) {
    const int64_t r = r0 + tid;
    int32_t src = -1, b = 0, len = 0;
    if (r < n) {
      src = perm ? perm[r] : (int32_t)r;
      b = rp[src];
      len = rp[src + 1] - b;
    }
    rb[tid] = b;
    rl[tid] = len;
    rs[tid] = src;
  }
  __syncthreads();
  const int32_t base = sptr[s];
  const int w = (sptr[s + 1] - base) / kSlice;
  for (int idx = tid; idx < kSlice * w; idx += kBlock) {
    const int row = idx / w, t = idx - row * w;
    int32_t c = 0;
    double v = 0.0;
    if (t < rl[row]) {
      const int32_t j = col[rb[row] + t];
      v = val[rb[row] + t];
      c = cmap ? cmap[j] : j;
      if (diag && j == rs[row]) diag[r0 + row] = v;
    }
    lc[row * pitch + t] = c;
    lv[row * pitch + t] = v;
  }
  __syncthreads();
  for (int idx = tid; idx < kSlice * w; idx += kBlock) {
    const int t = idx / kSlice, ln = idx - t * kSlice;
    const int64_t o = base + (int64_t)t * kSlice + ln;
    scol[o] = lc[ln * pitch + t];
    sval[o] = lv[ln * pitch + t];
  }
}

// *out = max(*out, max_i v[i] + add)
__global__ void __launch_bounds__(kBlock) k_max_i32(const int32_t* v, int64_t n, int32_t add, int32_t* out) {
  int32_t m = 0;
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBlock)
    m = v[i] + add > m ? v[i] + add : m;
  m = block_reduce(m, [](int32_t a, int32_t b) { return a > b ? a : b; });
  if (threadIdx.x == 0 && m) atomicMax(out, m);
}

void max_i32(const int32_t* v, int64_t n, int32_t add, int32_t* out, hipStream_t s) {
  k_max_i32<<<std::min(blocks_for(n), kReduceGrid), kBlock, 0, s>>>(v, n, add, out);
}

// nnz of colour class c = prefix[cptr[c+1]] - prefix[cptr[c]] of the row lengths
__global__ void k_color_nnz(const int32_t* prefix, const int32_t* cptr, int nc, int32_t* cnnz) {
  int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c < nc) cnnz[c] = prefix[cptr[c + 1]] - prefix[cptr[c]];
}

// P in the new numbering, SoA ELL-3 ([3][n]); padding repeats the first
// column with weight 0.
__global__ void k_p_layout(const int32_t* __restrict__ perm, const int32_t* __restrict__ ciperm,
                           const int32_t* __restrict__ pcol, const double* __restrict__ pval,
                           const int32_t* __restrict__ pcnt, int64_t n, int32_t* __restrict__ qcol,
                           double* __restrict__ qval, int32_t* __restrict__ qcnt) {
  int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n) return;
  const int32_t old = perm[r];
  const int32_t c = pcnt[old];
  int32_t pc[3], cc[3];
  double pv[3];
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    pc[t] = pcol[3 * old + t];
    pv[t] = pval[3 * old + t];
  }
#pragma unroll
  for (int t = 0; t < 3; ++t) cc[t] = t < c ? ciperm[pc[t]] : 0;
  qcnt[r] = c;
  const int32_t first = c > 0 ? cc[0] : 0;
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    qcol[t * n + r] = t < c ? cc[t] : first;
    qval[t * n + r] = t < c ? pv[t] : 0.0;
  }
}

// ------------------------------------------------------------------ coarsest level
__global__ void k_dense_scatter(const int32_t* rp, const int32_t* col, const double* val, int64_t n,
                                double* D) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  for (int32_t e = rp[i]; e < rp[i + 1]; ++e) D[i * n + col[e]] = val[e];
}

// Blocked dense Cholesky (32-column panels).  Entry (i, c) receives its updates
// -L[i][j] * L[c][j] one at a time in ascending j, then (below the diagonal)
// the division by L[c][c]: the same operations in the same order as the
// column-by-column definition, whatever the blocking.
constexpr int kPanel = 32;

// Lane l's value of v.
__device__ __forceinline__ double read_lane(double v, int l) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, l);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), l);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// One step of the factorisation, in one launch: the updates of panel j0 = k0 - 32
// (none at k0 = 0) to everything right of it, and the factorisation of panel k0.
// D holds the matrix with the updates of the panels before j0; the factor goes
// to L and, transposed, to U, so that no workgroup reads what another writes.
//
// The first `groups` workgroups each take 32 of the rows below the diagonal
// block of panel k0, and that block as well: all of them factor it alike, in
// wavefronts whose lanes 0-31 hold the rows of the block and lanes 32-63 the
// rows below.  Eight columns at a time: the first wavefront runs their chain of
// square root, division and first update (206 cycles a column), then the eight
// wavefronts update the columns to the right, a wavefront getting one double
// precision operation in 8 cycles.  The other workgroups update the tiles right
// of panel k0.  194 rows: 12.4 us a panel, of which the columns 8 us (the block
// in one wavefront, then the rows below it in registers, then the tiles in a
// second launch: 25 + 4.7 us).
constexpr int kCholT = 512;
__global__ void __launch_bounds__(kCholT) k_chol_step(double* __restrict__ D, int32_t n, int32_t k0, int32_t groups,
                                                      double* __restrict__ L, double* __restrict__ U,
                                                      int32_t* flags) {
  __shared__ double P[2 * kPanel][kPanel + 1];      // panel j0: rows of the group (or of the tile's two ranges)
  const int tid = threadIdx.x;
  const int32_t j0 = k0 - kPanel, kb = min(n - k0, kPanel);
  const bool first = k0 == 0;
  constexpr int kRows = kCholT / kPanel, kPer = 2 * kPanel / kRows, kSub = 8;
  const int cc = tid % kPanel, r0 = tid / kPanel;
  if ((int32_t)blockIdx.x < groups) {
    __shared__ double R[2 * kPanel][kPanel + 1];
    const int32_t below = k0 + kPanel + (int32_t)blockIdx.x * kPanel;   // first row below of this group
    auto row_of = [&](int r) { return r < kPanel ? k0 + r : below + r - kPanel; };
    double pv[kPer], dv[kPer];                     // all loads in flight together
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int64_t i = min(row_of(r0 + u * kRows), n - 1);
      pv[u] = first ? 0.0 : L[i * n + j0 + cc];
      dv[u] = D[i * n + min(k0 + cc, n - 1)];
    }
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int r = r0 + u * kRows;
      P[r][cc] = row_of(r) < n ? pv[u] : 0.0;
      const bool in = row_of(r) < n && cc < kb && (r >= kPanel || cc <= r);
      R[r][cc] = in ? dv[u] : (r == cc ? 1.0 : 0.0);   // past the matrix: the identity's columns
    }
    __syncthreads();
    // the updates of panel j0, four columns a wavefront
    const int lane = tid % kWave, w = tid / kWave;
    if (!first) {
      double a[kSub / 2];
#pragma unroll
      for (int u = 0; u < kSub / 2; ++u) a[u] = R[lane][w * (kSub / 2) + u];
#pragma unroll 4
      for (int j = 0; j < kPanel; ++j) {
        const double l = P[lane][j];
#pragma unroll
        for (int u = 0; u < kSub / 2; ++u) a[u] = a[u] - l * P[w * (kSub / 2) + u][j];
      }
#pragma unroll
      for (int u = 0; u < kSub / 2; ++u) R[lane][w * (kSub / 2) + u] = a[u];
      __syncthreads();
    }
    for (int g = 0; g < kb; g += kSub) {
      if (w == 0) {
        double r[kSub];
        bool ok = true;
#pragma unroll
        for (int u = 0; u < kSub; ++u) r[u] = R[lane][g + u];
#pragma unroll
        for (int u = 0; u < kSub; ++u) {
          const double dc = read_lane(r[u], g + u);
          ok = ok && dc > 0.0;
          const double d = ok ? sqrt(dc) : 1.0;
          r[u] = lane == g + u ? d : r[u] / d;
#pragma unroll
          for (int m = u + 1; m < kSub; ++m) r[m] = r[m] - r[u] * read_lane(r[u], g + m);
        }
#pragma unroll
        for (int u = 0; u < kSub; ++u) R[lane][g + u] = r[u];
        if (!ok && lane == 0 && blockIdx.x == 0) atomicOr(flags, F_NOT_SPD);
      }
      __syncthreads();
      double l[kSub];
#pragma unroll
      for (int u = 0; u < kSub; ++u) l[u] = R[lane][g + u];
#pragma unroll
      for (int t = 0; t < kPanel / kSub - 1; ++t) {
        const int c = g + kSub + w + t * (kCholT / kWave);
        if (c < kPanel) {
          double a = R[lane][c];
#pragma unroll
          for (int u = 0; u < kSub; ++u) a = a - l[u] * R[c][g + u];
          R[lane][c] = a;
        }
      }
      __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int r = r0 + u * kRows, i = row_of(r);
      if (i < n && cc < kb && (r >= kPanel || (blockIdx.x == 0 && cc <= r))) L[(int64_t)i * n + k0 + cc] = R[r][cc];
    }
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int c = w + u * (kCholT / kWave), i = row_of(lane);
      if (i < n && c < kb && (lane >= kPanel || (blockIdx.x == 0 && c <= lane))) U[(int64_t)(k0 + c) * n + i] = R[lane][c];
    }
    return;
  }
  // a_ic <- a_ic - l_ij l_cj for the columns j of panel j0: tile (I, C) of the lower triangle
  int32_t t = (int32_t)blockIdx.x - groups, I = 0;
  while (t > I) t -= ++I;
  const int32_t ri = k0 + kPanel + I * kPanel, rc = k0 + kPanel + t * kPanel;
  double pv[kPer], a[kPer / 2];
  const int32_t c = rc + cc;
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int r = r0 + u * kRows;
    pv[u] = L[(int64_t)min(r < kPanel ? ri + r : rc + r - kPanel, n - 1) * n + j0 + cc];
    if (u < kPer / 2) a[u] = D[(int64_t)min(ri + r, n - 1) * n + min(c, n - 1)];
  }
#pragma unroll
  for (int u = 0; u < kPer; ++u) P[r0 + u * kRows][cc] = pv[u];
  __syncthreads();
#pragma unroll 4
  for (int j = 0; j < kPanel; ++j) {
    const double l = P[kPanel + cc][j];
#pragma unroll
    for (int u = 0; u < kPer / 2; ++u) a[u] = a[u] - P[r0 + u * kRows][j] * l;
  }
#pragma unroll
  for (int u = 0; u < kPer / 2; ++u) {
    const int32_t i = ri + r0 + u * kRows;
    if (i < n && c <= i) D[(int64_t)i * n + c] = a[u];
  }
}

// Column c of the coarsest inverse, A^-1 e_c, by substitution with the
// factor: forward L y = e_c, row i subtracting L_ik y_k for k ascending, then
// back L^T x = y, row i subtracting L_ki x_k for k descending from n - 1; each
// row is then divided by its pivot.  Both run column-oriented: once y_k (x_k)
// is known, every row that needs it subtracts its term, so each row performs
// its subtractions in the order of the row-by-row definition, bit for bit.
// Rows above c start at +0 and stay +0 (every term they would subtract is a
// product with y_k = +0), so the forward pass starts at row c.
//
// One wavefront per column: lane l holds rows l, l + 64, ... (S slots) in
// registers, with their pivots, and the pivot row's value is read across lanes;
// the factor entries of the next D steps are loaded ahead (phase k mod D of a
// ring).  What bounds a column is its chain, a division, a product and a
// difference per step (130 cycles), as long as no step waits for a load: the
// loads are therefore issued without conditions, past the last row those of the
// last row again (loads under conditions had the compiler wait for the newest
// one, and a pivot loaded as a scalar for all: 450 cycles a step; 194 rows: 88 us,
// now 43; 513-768 rows: 484, now 237; 1000 rows: 907, now 428).
//
// U holds the factor's columns from the diagonal on and nothing before it: row k of U
// left of column k is not written.  The forward pass reads those entries, within the
// pivot's own slot, and drops what it makes of them (rows up to k keep their values).
template <class F, int... Q>
__device__ __forceinline__ void each_slot_of(F&& f, std::integer_sequence<int, Q...>) {
  (f(std::integral_constant<int, Q>{}), ...);
}
template <int S, class F>
__device__ __forceinline__ void each_slot(F&& f) {
  each_slot_of(f, std::make_integer_sequence<int, S>{});
}

template <int S, int D>
__global__ void __launch_bounds__(kWave) k_coarse_inverse(const double* __restrict__ L,
                                                         const double* __restrict__ U, int32_t n,
                                                         double* __restrict__ inv) {
  const int32_t c = blockIdx.x;
  const int lane = threadIdx.x;
  double s[S], d[S], f[D][S];                 // f: factor entries of step k at phase k mod D
  int32_t at[S];                              // the slots' rows (past the end: the last row)
#pragma unroll
  for (int q = 0; q < S; ++q) {
    at[q] = min(q * kWave + lane, n - 1);
    s[q] = q * kWave + lane == c ? 1.0 : 0.0;
    d[q] = L[(int64_t)at[q] * n + at[q]];
  }
  // forward: step k uses column k of L (row k of U) for rows i > k
  const int32_t k_first = c - c % D;
#pragma unroll
  for (int j = 0; j < D; ++j)
#pragma unroll
    for (int q = 0; q < S; ++q) f[j][q] = U[(int64_t)min(k_first + j, n - 1) * n + at[q]];
  each_slot<S>([&](auto Q) {
    constexpr int q = Q;
    const int32_t k_hi = min(n, (q + 1) * kWave);
    for (int32_t k0 = max(k_first, q * kWave); k0 < k_hi; k0 += D) {
#pragma unroll
      for (int j = 0; j < D; ++j) {
        const int32_t k = k0 + j;
        if (k >= c && k < n) {
          const double y = read_lane(s[q], k & (kWave - 1)) / read_lane(d[q], k & (kWave - 1));
          const double t = s[q] - f[j][q] * y;
          const int32_t i = q * kWave + lane;
          s[q] = i > k ? t : (i == k ? y : s[q]);
#pragma unroll
          for (int q2 = q + 1; q2 < S; ++q2) s[q2] = s[q2] - f[j][q2] * y;
        }
        const double* __restrict__ row = U + (int64_t)min(k + D, n - 1) * n;
#pragma unroll
        for (int q2 = q; q2 < S; ++q2) f[j][q2] = row[at[q2]];
      }
    }
  });
  // back: step i uses row i of L for rows r < i (rows past the end hold no row's value)
  const int32_t i_first = n - 1 + (D - 1 - (n - 1) % D);
#pragma unroll
  for (int j = 0; j < D; ++j)
#pragma unroll
    for (int q = 0; q < S; ++q) f[j][q] = L[(int64_t)min(i_first - (D - 1) + j, n - 1) * n + at[q]];
  each_slot<S>([&](auto Q) {
    constexpr int q = S - 1 - Q;
    // groups of D steps aligned to multiples of D, top step i0 first
    for (int32_t i0 = min(i_first, (q + 1) * kWave - 1); i0 >= q * kWave; i0 -= D) {
#pragma unroll
      for (int j = D - 1; j >= 0; --j) {
        const int32_t i = i0 - (D - 1) + j;
        if (i < n) {
          const double x = read_lane(s[q], i & (kWave - 1)) / read_lane(d[q], i & (kWave - 1));
          const double t = s[q] - f[j][q] * x;
          const int32_t r = q * kWave + lane;
          s[q] = r < i ? t : (r == i ? x : s[q]);
#pragma unroll
          for (int q2 = 0; q2 < q; ++q2) s[q2] = s[q2] - f[j][q2] * x;
        }
        const double* __restrict__ row = L + (int64_t)max(i - D, 0) * n;
#pragma unroll
        for (int q2 = 0; q2 <= q; ++q2) f[j][q2] = row[at[q2]];
      }
    }
  });
  const int32_t ld = (int32_t)inv_ld(n);
#pragma unroll
  for (int q = 0; q < S; ++q) {
    const int32_t i = q * kWave + lane;
    if (i < ld) inv[(int64_t)c * ld + i] = i < n ? s[q] : 0.0;
  }
}

// The same operations for coarsest levels beyond the register form: the
// column lives in LDS, one workgroup per column, a barrier per step.
__global__ void __launch_bounds__(kBlock) k_coarse_inverse_lds(const double* __restrict__ L,
                                                               const double* __restrict__ U, int32_t n,
                                                               double* __restrict__ inv) {
  extern __shared__ double col[];
  const int32_t c = blockIdx.x;
  for (int32_t i = threadIdx.x; i < n; i += kBlock) col[i] = i == c ? 1.0 : 0.0;
  __syncthreads();
  for (int32_t k = c; k < n; ++k) {
    const double y = col[k] / L[(int64_t)k * n + k];
    for (int32_t i = k + 1 + threadIdx.x; i < n; i += kBlock) col[i] = col[i] - U[(int64_t)k * n + i] * y;
    __syncthreads();                          // every thread has read col[k]
    if (threadIdx.x == 0) col[k] = y;
    __syncthreads();
  }
  for (int32_t i = n - 1; i >= 0; --i) {
    const double x = col[i] / L[(int64_t)i * n + i];
    for (int32_t r = threadIdx.x; r < i; r += kBlock) col[r] = col[r] - L[(int64_t)i * n + r] * x;
    __syncthreads();
    if (threadIdx.x == 0) col[i] = x;
    __syncthreads();
  }
  const int32_t ld = (int32_t)inv_ld(n);
  for (int32_t i = threadIdx.x; i < ld; i += kBlock) inv[(int64_t)c * ld + i] = i < n ? col[i] : 0.0;
}

// ------------------------------------------------------------------ block order
// Order-preserving 64-bit key of a double (a larger double gets a larger
// key), so that minima and maxima are exact integer atomics.
__device__ __forceinline__ unsigned long long ordered_key(double v) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
  return (u >> 63) ? ~u : (u | (1ull << 63));
}

__global__ void k_grid_keys_init(unsigned long long* keys) {
  const int i = threadIdx.x;
  if (i < 9) keys[i] = i < 3 ? ~0ull : 0ull;
}

// keys[0..2]: minima and keys[3..5]: maxima of the three coordinates (ordered
// keys); keys[6..8]: largest |X_j,a - X_i,a| over the stored off-diagonal
// entries (i, j) of A_l, per axis a (non-negative doubles, whose bit patterns
// order as integers).
__global__ void __launch_bounds__(kBlock) k_grid_extents(const double* __restrict__ X, const int32_t* __restrict__ rp,
                                                         const int32_t* __restrict__ col, int64_t n,
                                                         unsigned long long* keys) {
  unsigned long long mn[3] = {~0ull, ~0ull, ~0ull}, mx[3] = {0, 0, 0}, dm[3] = {0, 0, 0};
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBlock) {
    const double xi[3] = {X[3 * i], X[3 * i + 1], X[3 * i + 2]};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const unsigned long long k = ordered_key(xi[a]);
      mn[a] = k < mn[a] ? k : mn[a];
      mx[a] = k > mx[a] ? k : mx[a];
    }
    for (int32_t e = rp[i]; e < rp[i + 1]; ++e) {
      const int64_t j = col[e];
      if (j == i) continue;
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const unsigned long long d = __builtin_bit_cast(unsigned long long, fabs(X[3 * j + a] - xi[a]));
        dm[a] = d > dm[a] ? d : dm[a];
      }
    }
  }
  auto lo = [](unsigned long long u, unsigned long long v) { return u < v ? u : v; };
  auto hi = [](unsigned long long u, unsigned long long v) { return u > v ? u : v; };
  unsigned long long r[9];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    r[a] = block_reduce(mn[a], lo);
    __syncthreads();
    r[3 + a] = block_reduce(mx[a], hi);
    __syncthreads();
    r[6 + a] = block_reduce(dm[a], hi);
    __syncthreads();
  }
  if (threadIdx.x == 0) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      atomicMin(&keys[a], r[a]);
      atomicMax(&keys[3 + a], r[3 + a]);
      atomicMax(&keys[6 + a], r[6 + a]);
    }
  }
}

// Colour of brick bx of cell row cy: with a = bx - (cy + 1) div 2, (a - cy)
// mod 3.  A brick holds the cells cx of its row with (cx + cy mod 2) div 2 =
// bx (two cells side by side, shifted by one cell on odd rows); it touches
// two bricks in its row and two in each neighbouring row, and these six
// colours all differ from its own.
__host__ __device__ inline int32_t brick_color(int64_t bx, int64_t cy) {
  const int64_t a = bx - (cy + 1) / 2;
  return (int32_t)(((a - cy) % 3 + 3) % 3);
}

// Block colour of block id c (bricks: cy nbx + bx with nbx = gx div 2 + 1;
// single cells: cy gx + cx, coloured by their parity pair).
__host__ __device__ inline int32_t block_color_of(int32_t c, int32_t gx, bool bricks) {
  if (bricks) {
    const int32_t nbx = gx / 2 + 1;
    return brick_color(c % nbx, c / nbx);
  }
  return (c % gx & 1) + 2 * (c / gx & 1);
}

// Brick (cy nbx + bx) and cell (cy gx + cx) of every point.
__global__ void k_grid_cells(const double* __restrict__ X, int64_t n, int a0, int a1, double lo0, double lo1,
                             double side, int32_t gx, int32_t* brick, int32_t* cell) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int64_t cx = (int64_t)floor((X[3 * i + a0] - lo0) / side);
  const int64_t cy = (int64_t)floor((X[3 * i + a1] - lo1) / side);
  brick[i] = (int32_t)(cy * (gx / 2 + 1) + (cx + (cy & 1)) / 2);
  cell[i] = (int32_t)(cy * gx + cx);
}

// The chosen blocks of every point and their colours.
__global__ void k_block_ids(const int32_t* brick, const int32_t* cell, int64_t n, int32_t gx, int32_t bricks,
                            int32_t* bcell, int32_t* bcolor) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int32_t c = bricks ? brick[i] : cell[i];
  bcell[i] = c;
  bcolor[i] = block_color_of(c, gx, bricks != 0);
}

// Sweep class of a row: block colour, then colour.
__global__ void k_sweep_class(const int32_t* bcolor, const int32_t* color, int64_t n, int32_t C, int32_t* cls) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) cls[i] = bcolor[i] * C + color[i];
}

__global__ void k_count_cells(const int32_t* bcell, int64_t n, int32_t* cnt) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool on = i < n;
  run_add(cnt, on ? bcell[i] : -1, on);
}

// Rows per brick and rows per cell, in one pass.
__global__ void k_count_cells2(const int32_t* brick, const int32_t* cell, int64_t n, int32_t* cntb, int32_t* cntc) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool on = i < n;
  run_add(cntb, on ? brick[i] : -1, on);
  run_add(cntc, on ? cell[i] : -1, on);
}

// ---- per-cell colouring of a level swept in block order (DSATUR in each cell)
constexpr int32_t kMaxCellRows = 512;     // larger blocks send the level back to the colour order
constexpr int32_t kMaxBrickRows = 256;    // a larger brick makes single cells the level's blocks
constexpr int32_t kMaxCellColors = 64;    // likewise a cell that needs this many colours
constexpr int32_t kCellAdjLds = 4096;     // in-cell couplings of a cell kept in LDS (else in HBM)

__global__ void k_cell_slots(const int32_t* bcell, int64_t n, int32_t* cnt, int32_t* slot) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool on = i < n;
  const int32_t t = run_add(cnt, on ? bcell[i] : -1, on);
  if (on) slot[i] = t;
}

__global__ void k_cell_scatter(const int32_t* __restrict__ bcell, int64_t n, const int32_t* __restrict__ cptr,
                               const int32_t* __restrict__ slot, int32_t* __restrict__ rows) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) rows[cptr[bcell[i]] + slot[i]] = (int32_t)i;
}

// The largest value over the wavefront, in every lane: running maxima within
// each row of 16 lanes (DPP row shifts by 1, 2, 4, 8; lanes shifted in from
// outside the row contribute 0), the row maxima carried across rows (DPP row
// broadcasts of lanes 15 and 31), then lane 63's value read back.
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
  auto mx = [](uint32_t a, uint32_t b) { return a > b ? a : b; };
  v = mx(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false));   // row_shr:1
  v = mx(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false));   // row_shr:2
  v = mx(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false));   // row_shr:4
  v = mx(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false));   // row_shr:8
  v = mx(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false));   // row_bcast:15
  v = mx(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false));   // row_bcast:31
  return (uint32_t)__builtin_amdgcn_readlane((int)v, kWave - 1);
}

// In-cell degree of row i (couplings to other rows of its cell), and the
// cell's total.
__global__ void k_incell_degree(const int32_t* __restrict__ arp, const int32_t* __restrict__ acol,
                                const int32_t* __restrict__ bcell, int64_t n, int32_t* __restrict__ deg,
                                int32_t* __restrict__ cell_deg) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool on = i < n;
  const int32_t c = on ? bcell[i] : -1;
  int32_t d = 0;
  if (on) {
    for (int32_t e = arp[i]; e < arp[i + 1]; ++e) {
      const int32_t j = acol[e];
      d += (j != (int32_t)i && bcell[j] == c) ? 1 : 0;
    }
    deg[i] = d;
  }
  run_sum(cell_deg, c, d, on);                 // one atomic per run of rows of one block
}

// DSATUR in one cell, one wavefront per cell.  The cell's rows are sorted
// ascending in LDS (bitonic), so a row's position is its rank by index; its
// in-cell neighbours become positions (binary search), kept in LDS when they
// fit and otherwise in the cell's segment of adj.  Each step colours the
// uncoloured row of largest saturation (distinct colours among its coloured
// in-cell neighbours), then largest in-cell degree, then smallest position,
// with the smallest colour none of its neighbours has.  A row that would need
// colour kMaxCellColors sets *overflow.
__global__ void __launch_bounds__(kWave) k_cell_dsatur(const int32_t* __restrict__ cptr,
                                                      const int32_t* __restrict__ rows,
                                                      const int32_t* __restrict__ deg_of,
                                                      const int32_t* __restrict__ cadj,
                                                      const int32_t* __restrict__ arp,
                                                      const int32_t* __restrict__ acol,
                                                      const int32_t* __restrict__ bcell, int32_t* __restrict__ adj,
                                                      int32_t* __restrict__ color, int32_t* __restrict__ maxcol,
                                                      int32_t* __restrict__ overflow) {
  __shared__ uint64_t mask[kMaxCellRows];
  __shared__ int32_t r[kMaxCellRows], deg[kMaxCellRows], off[kMaxCellRows + 1];
  __shared__ int32_t ladj[kCellAdjLds];
  const int32_t c = blockIdx.x;
  const int32_t base = cptr[c], m = cptr[c + 1] - base;
  if (m <= 0 || m > kMaxCellRows) return;
  const int lane = threadIdx.x;
  int32_t M = 1;
  while (M < m) M <<= 1;
  for (int32_t p = lane; p < M; p += kWave) r[p] = p < m ? rows[base + p] : INT32_MAX;
  __syncthreads();
  for (int32_t k = 2; k <= M; k <<= 1)
    for (int32_t j = k >> 1; j > 0; j >>= 1) {
      for (int32_t p = lane; p < M; p += kWave) {
        const int32_t q = p ^ j;
        if (q > p) {
          const int32_t x = r[p], y = r[q];
          if ((x > y) == ((p & k) == 0)) {
            r[p] = y;
            r[q] = x;
          }
        }
      }
      __syncthreads();
    }
  for (int32_t p = lane; p < m; p += kWave) {
    mask[p] = 0;
    deg[p] = deg_of[r[p]];
  }
  __syncthreads();
  if (lane == 0) {
    int32_t acc = 0;
    for (int32_t p = 0; p < m; ++p) {
      off[p] = acc;
      acc += deg[p];
    }
    off[m] = acc;
  }
  __syncthreads();
  int32_t* A = off[m] <= kCellAdjLds ? ladj : adj + cadj[c];
  for (int32_t p = lane; p < m; p += kWave) {
    const int32_t i = r[p];
    int32_t t = off[p];
    for (int32_t e = arp[i]; e < arp[i + 1]; ++e) {
      const int32_t j = acol[e];
      if (j == i || bcell[j] != c) continue;
      int32_t lo = 0, hi = m;
      while (lo < hi) {
        const int32_t mid = (lo + hi) >> 1;
        if (r[mid] < j) lo = mid + 1;
        else hi = mid;
      }
      A[t++] = lo;
    }
  }
  __threadfence_block();
  __syncthreads();
  // Lane l holds rows l + 64 q: their colour (-1: not yet coloured; rows past
  // m count as coloured) and degree in registers, so a step reads only the
  // rows' masks from LDS, all of them at once.
  constexpr int kQ = kMaxCellRows / kWave;
  int32_t cq[kQ], dq[kQ];
#pragma unroll
  for (int q = 0; q < kQ; ++q) {
    const int32_t p = lane + q * kWave;
    cq[q] = p < m ? -1 : 0;
    dq[q] = p < m ? deg[p] : 0;
  }
  int32_t used = 0;
  for (int32_t step = 0; step < m; ++step) {
    uint64_t mk[kQ];
#pragma unroll
    for (int q = 0; q < kQ; ++q) mk[q] = mask[lane + q * kWave];
    uint32_t best = 0;
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
      const int32_t p = lane + q * kWave;
      const uint32_t key = ((uint32_t)__popcll(mk[q]) << 20) | ((uint32_t)dq[q] << 10) | (uint32_t)(1023 - p);
      best = cq[q] < 0 && key > best ? key : best;
    }
    best = wave_max_u32(best);
    const int32_t v = 1023 - (int32_t)(best & 1023u);
    const uint64_t free_colours = ~mask[v];
    if (free_colours == 0) {                // every colour below kMaxCellColors is taken
      if (lane == 0) atomicOr(overflow, 1);
      return;
    }
    const int32_t k = __builtin_ctzll(free_colours);
    used = used > k ? used : k;
#pragma unroll
    for (int q = 0; q < kQ; ++q)
      if (lane + q * kWave == v) cq[q] = k;
    __syncthreads();
    for (int32_t t = lane; t < deg[v]; t += kWave) mask[A[off[v] + t]] |= uint64_t(1) << k;
    __syncthreads();
  }
#pragma unroll
  for (int q = 0; q < kQ; ++q) {
    const int32_t p = lane + q * kWave;
    if (p < m) color[r[p]] = cq[q];
  }
  if (lane == 0) atomicMax(maxcol, used);
}

// Slot v of the block numbering, [0, 4 H) with H block ids: id v mod H if its
// colour is k = v div H (else -1); blocks are numbered by colour, then id.
__device__ __forceinline__ int32_t grid_cell_of(int64_t v, int64_t H, int32_t gx, bool bricks) {
  const int32_t k = (int32_t)(v / H);
  const int32_t b = (int32_t)(v % H);
  return block_color_of(b, gx, bricks) == k ? b : -1;
}

__global__ void k_cell_flags(const int32_t* cnt, int64_t H, int32_t gx, int32_t bricks, int32_t* flag) {
  const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= 4 * H) return;
  const int32_t c = grid_cell_of(v, H, gx, bricks != 0);
  flag[v] = c >= 0 && cnt[c] > 0 ? 1 : 0;
}

// Block (compact id) of every solve row.
__global__ void k_row_block(const int32_t* perm, const int32_t* bcell, int64_t n, const int32_t* vid, int64_t H,
                            int32_t gx, int32_t bricks, int32_t* blk) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= n) return;
  const int32_t c = bcell[perm[g]];
  blk[g] = vid[(int64_t)block_color_of(c, gx, bricks != 0) * H + c];
}

// First local row of every colour c = 0..C in every block (rows of a block are
// ascending solve rows, so ascending colours).
__global__ void k_block_cls(const int32_t* boff, const int32_t* brows, const int32_t* perm, const int32_t* color,
                            int32_t nblk, int32_t C, int32_t* bcls) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (int64_t)nblk * (C + 1)) return;
  const int32_t b = (int32_t)(t / (C + 1)), c = (int32_t)(t % (C + 1));
  int32_t lo = boff[b], hi = boff[b + 1];
  const int32_t base = lo;
  while (lo < hi) {
    const int32_t mid = (lo + hi) >> 1;
    if (color[perm[brows[mid]]] < c) lo = mid + 1; else hi = mid;
  }
  bcls[t] = lo - base;
}

// Per local row: its length (entries of A_l, diagonal included) and colour,
// packed as len << 8 | colour; per block: the mask of its colours.
__global__ void k_block_rowinfo(const int32_t* rp, const int32_t* perm, const int32_t* color, const int32_t* brows,
                                int64_t n, int32_t* rinfo) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const int32_t o = perm[brows[k]];
  rinfo[k] = ((rp[o + 1] - rp[o]) << 8) | color[o];
}

// Per block: its header and its gather list (own rows, then halo rows, padded with the
// block's first row, so that loads of padding slots share a line with a real load).
__global__ void k_block_gather(const int32_t* boff, const int32_t* brows, const int32_t* hoff, const int32_t* hlist,
                               const int32_t* bw, const int32_t* beoff, const uint64_t* bmask, int32_t gstride,
                               BlockHdr* hdr, int32_t* glist) {
  const int32_t b = blockIdx.x;
  const int32_t r0 = boff[b], rows = boff[b + 1] - r0, h0 = hoff[b], nh = hoff[b + 1] - h0;
  if (threadIdx.x == 0) {
    BlockHdr hd;
    hd.r0 = r0;
    hd.rows = rows;
    hd.nh = nh;
    hd.w = bw[b];
    hd.e0 = beoff[b];
    hd.pad = 0;
    hd.mask = bmask[b];
    hdr[b] = hd;
  }
  for (int32_t k = threadIdx.x; k < gstride; k += blockDim.x)
    glist[(int64_t)b * gstride + k] = k < rows ? brows[r0 + k] : (k < rows + nh ? hlist[h0 + k - rows] : brows[r0]);
}

__global__ void k_block_mask(const int32_t* bcls, int32_t nblk, int32_t C, uint64_t* bmask) {
  const int32_t b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= nblk) return;
  uint64_t m = 0;
  for (int32_t c = 0; c < C; ++c)
    if (bcls[(int64_t)b * (C + 1) + c] < bcls[(int64_t)b * (C + 1) + c + 1]) m |= uint64_t(1) << c;
  bmask[b] = m;
}


__global__ void k_block_cells(const int32_t* boff, const int32_t* bw, int32_t nblk, int32_t* sz) {
  const int32_t b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b < nblk) sz[b] = bw[b] * (boff[b + 1] - boff[b]);
}

// The halo of every block, one workgroup per block: the rows of other blocks
// that its rows read, collected in LDS, sorted (bitonic) and kept once each,
// written at the block's slot base tmp + tcap[b] (capacity: its entries);
// hcnt[b] receives their number.  A coupling to another block of the same
// block colour (which the grid excludes), or more than kHaloSort collected
// entries, raises *bad.
constexpr int kHaloSort = 4096;
__global__ void __launch_bounds__(kBlock) k_block_halo(const int32_t* __restrict__ rp, const int32_t* __restrict__ col,
                                                       const int32_t* __restrict__ perm,
                                                       const int32_t* __restrict__ iperm,
                                                       const int32_t* __restrict__ blk,
                                                       const int32_t* __restrict__ bcolor,
                                                       const int32_t* __restrict__ boff,
                                                       const int32_t* __restrict__ brows, int32_t* tmp,
                                                       const int32_t* __restrict__ tcap, int32_t* hcnt, int32_t* bad) {
  __shared__ int32_t a[kHaloSort];
  __shared__ int32_t part[kBlock + 1];
  __shared__ int32_t na;
  const int32_t b = blockIdx.x;
  const int32_t r0 = boff[b], rows = boff[b + 1] - r0;
  if (threadIdx.x == 0) na = 0;
  __syncthreads();
  for (int32_t p = threadIdx.x; p < rows; p += kBlock) {
    const int32_t g = brows[r0 + p], o = perm[g];
    for (int32_t e = rp[o]; e < rp[o + 1]; ++e) {
      const int32_t oc = col[e];
      if (oc == o) continue;
      const int32_t j = iperm[oc];
      if (blk[j] == b) continue;
      if (bcolor[oc] == bcolor[o]) atomicOr(bad, 1);
      const int32_t k = atomicAdd(&na, 1);
      if (k < kHaloSort) a[k] = j;
    }
  }
  __syncthreads();
  const int32_t len = na;
  if (len > kHaloSort) {
    if (threadIdx.x == 0) {
      atomicOr(bad, 2);
      hcnt[b] = 0;
    }
    return;
  }
  int32_t P = 1;
  while (P < len) P <<= 1;
  for (int32_t i = len + threadIdx.x; i < P; i += kBlock) a[i] = INT32_MAX;
  __syncthreads();
  for (int32_t k = 2; k <= P; k <<= 1)
    for (int32_t j = k >> 1; j > 0; j >>= 1) {
      for (int32_t i = threadIdx.x; i < P; i += kBlock) {
        const int32_t l = i ^ j;
        if (l > i) {
          const bool up = (i & k) == 0;
          const int32_t x = a[i], y = a[l];
          if ((x > y) == up) {
            a[i] = y;
            a[l] = x;
          }
        }
      }
      __syncthreads();
    }
  // distinct values: each thread counts the first occurrences in its chunk
  const int32_t chunk = (len + kBlock - 1) / kBlock;
  const int32_t c0 = threadIdx.x * chunk, c1 = min(len, c0 + chunk);
  int32_t cnt = 0;
  for (int32_t i = c0; i < c1; ++i) cnt += (i == 0 || a[i] != a[i - 1]) ? 1 : 0;
  part[threadIdx.x + 1] = cnt;
  __syncthreads();
  if (threadIdx.x == 0) {
    part[0] = 0;
    for (int t = 1; t <= kBlock; ++t) part[t] += part[t - 1];
    hcnt[b] = part[kBlock];
  }
  __syncthreads();
  int32_t w = tcap[b] + part[threadIdx.x];
  for (int32_t i = c0; i < c1; ++i)
    if (i == 0 || a[i] != a[i - 1]) tmp[w++] = a[i];
}

// Entries of A_l (diagonal included) in the rows of every block: the halo's capacity.
// Entries (cap) and longest row (bw) of every block, a wavefront per block.
__global__ void k_block_entries(const int32_t* rp, const int32_t* perm, const int32_t* brows, const int32_t* boff,
                                int32_t nblk, int32_t* cap, int32_t* bw) {
  const int32_t b = (int32_t)(((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave);
  if (b >= nblk) return;
  int32_t s = 0, w = 0;
  for (int32_t k = boff[b] + (int32_t)(threadIdx.x & (kWave - 1)); k < boff[b + 1]; k += kWave) {
    const int32_t o = perm[brows[k]];
    const int32_t len = rp[o + 1] - rp[o];
    s += len;
    w = max(w, len);
  }
  s = wave_sum(s);
  for (int o = kWave / 2; o > 0; o >>= 1) w = max(w, __shfl_xor(w, o, kWave));
  if ((threadIdx.x & (kWave - 1)) == 0) {
    cap[b] = s;
    bw[b] = w;
  }
}

// The block ELL, one workgroup per block (its halo in LDS), kEllLanes lanes a
// row (a row's entries each take four dependent loads: 143,637 rows 62 us with
// one lane, now 45): entry t of local
// row p of block b at beoff[b] + t rows_b + p; the LDS slot of its column
// (own row: its local row; another block's row: rows_b + its position in the
// block's halo) and its value; the diagonal and the padding up to the block's
// width point at the zero slot rows_b + halo_b with value 0.
constexpr int kEllLanes = 16;
__global__ void __launch_bounds__(kBlock) k_block_ell(const int32_t* __restrict__ rp, const int32_t* __restrict__ col,
                                                      const double* __restrict__ val, const int32_t* __restrict__ perm,
                                                      const int32_t* __restrict__ iperm,
                                                      const int32_t* __restrict__ blk,
                                                      const int32_t* __restrict__ lpos,
                                                      const int32_t* __restrict__ boff,
                                                      const int32_t* __restrict__ brows,
                                                      const int32_t* __restrict__ hoff,
                                                      const int32_t* __restrict__ hlist,
                                                      const int32_t* __restrict__ bw,
                                                      const int32_t* __restrict__ beoff, int32_t* elx, double* elv) {
  __shared__ int32_t hl[kHaloSort];
  const int32_t b = (int32_t)xcd_block();
  const int32_t r0 = boff[b], rows = boff[b + 1] - r0;
  const int32_t h0 = hoff[b], nh = hoff[b + 1] - h0;
  for (int32_t k = threadIdx.x; k < nh; k += kBlock) hl[k] = hlist[h0 + k];
  __syncthreads();
  const int32_t pad = rows + nh, w = bw[b], e0 = beoff[b];
  for (int32_t p = threadIdx.x / kEllLanes; p < rows; p += kBlock / kEllLanes) {
    const int32_t o = perm[brows[r0 + p]];
    const int32_t rb = rp[o], len = rp[o + 1] - rb;
    for (int32_t t = threadIdx.x % kEllLanes; t < w; t += kEllLanes) {
      int32_t slot = pad;
      double v = 0.0;
      if (t < len) {
        const int32_t oc = col[rb + t];
        if (oc != o) {
          const int32_t j = iperm[oc];
          if (blk[j] == b) {
            slot = lpos[j];
          } else {
            int32_t lo = 0, hi = nh;
            while (lo < hi) {
              const int32_t mid = (lo + hi) >> 1;
              if (hl[mid] < j) lo = mid + 1; else hi = mid;
            }
            slot = rows + lo;
          }
          v = val[rb + t];
        }
      }
      elx[e0 + t * rows + p] = slot;
      elv[e0 + t * rows + p] = v;
    }
  }
}

// Local row of every solve row: its position in the block's row list.
__global__ void k_local_rows(const int32_t* bpos, const int32_t* blk, const int32_t* boff, int64_t n, int32_t* lpos) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g < n) lpos[g] = bpos[g] - boff[blk[g]];
}

// mx[0] = most rows, mx[1] = longest halo, mx[2] = widest ELL of any block, mx[3] and
// mx[4] = most LDS of a block in the batched sweep (mblock_layout), in float and double.
__global__ void __launch_bounds__(kBlock) k_block_maxima(const int32_t* boff, const int32_t* hoff, const int32_t* bw,
                                                         int32_t nblk, int32_t C, int32_t* mx) {
  int32_t r = 0, hl = 0, w = 0, l4 = 0, l8 = 0;
  for (int32_t b = blockIdx.x * kBlock + threadIdx.x; b < nblk; b += gridDim.x * kBlock) {
    r = max(r, boff[b + 1] - boff[b]);
    hl = max(hl, hoff[b + 1] - hoff[b]);
    w = max(w, bw[b]);
    const int32_t rows = boff[b + 1] - boff[b], nh = hoff[b + 1] - hoff[b];
    l4 = max(l4, mblock_layout(rows, nh, bw[b], C, 4).bytes);
    l8 = max(l8, mblock_layout(rows, nh, bw[b], C, 8).bytes);
  }
  auto mxop = [](int32_t a, int32_t b) { return a > b ? a : b; };
  r = block_reduce(r, mxop);
  __syncthreads();
  hl = block_reduce(hl, mxop);
  __syncthreads();
  w = block_reduce(w, mxop);
  __syncthreads();
  l4 = block_reduce(l4, mxop);
  __syncthreads();
  l8 = block_reduce(l8, mxop);
  if (threadIdx.x == 0) {
    atomicMax(&mx[3], l4);
    atomicMax(&mx[4], l8);
    atomicMax(&mx[0], r);
    atomicMax(&mx[1], hl);
    atomicMax(&mx[2], w);
  }
}

constexpr int32_t kMaxBlocks = 8192;         // blocks of a level (the partition's LDS histogram)
constexpr int64_t kBlkLdsMax = 64 * 1024;    // LDS of a block sweep (its rows, halo and zero slot)

// New values of A_l into the block ELL (same slots).
__global__ void k_block_values(const int32_t* rp, const int32_t* col, const double* val, const int32_t* perm,
                               const int32_t* boff, const int32_t* brows, const int32_t* bw, const int32_t* beoff,
                               int32_t nblk, double* elv) {
  const int32_t b = blockIdx.x;
  if (b >= nblk) return;
  const int32_t r0 = boff[b], rows = boff[b + 1] - r0, w = bw[b], e0 = beoff[b];
  for (int32_t p = threadIdx.x / kEllLanes; p < rows; p += kBlock / kEllLanes) {
    const int32_t o = perm[brows[r0 + p]];
    const int32_t rb = rp[o], len = rp[o + 1] - rb;
    for (int32_t t = threadIdx.x % kEllLanes; t < w; t += kEllLanes)
      elv[e0 + t * rows + p] = t < len && col[rb + t] != o ? val[rb + t] : 0.0;
  }
}
}  // namespace

// Jones-Plassmann colouring takes tens of rounds on the Galerkin levels (about
// the degree): the host checks the worklist every kColorBatch rounds.
constexpr int kColorBatch = 16;

void colouring(Handle& h, Level& lv, int level) {
  hipStream_t s = h.stream;
  int64_t n = lv.n;
  lv.color = (int32_t*)dalloc(h, (size_t)n * 4);
  fill_i32(lv.color, -1, n, s);
  int32_t* ncol = (int32_t*)talloc(s, 4);
  ColorKey key{(h.opt.seed ^ kColorSalt) ^ ((uint64_t)level << 32)};
  int32_t* wl = (int32_t*)talloc(s, (size_t)2 * n * 4);
  ColorLists L;
  if (n <= kColorListLevel) {
    L.list = (int32_t*)talloc(s, (size_t)n * kColorList * 4);
    L.mask = (uint64_t*)talloc(s, (size_t)n * 8);
    L.cnt = (uint8_t*)talloc(s, (size_t)n);
  }
  const int grid = std::min(blocks_for(n), 4 * kRoundGrid);
  int k = 0;
  const int64_t lds_small = small_color_lds(n, lv.nnzA);
  if (n <= kSmallColorRows && lds_small <= kSmallColorLds) {
    // the whole level, passes included, in one workgroup
    k_color_small<<<1, kDrainItems, (size_t)lds_small, s>>>(lv.arp, lv.acol, (int32_t)n, key, h.opt.color_passes,
                                                            lv.color, ncol, h.flags);
    int64_t nco = 0, fl = 0;
    ScalarRead rd[2] = {{ncol, 4, &nco}, {h.flags, 4, &fl}};
    read_scalars(h, rd, 2);
    if (fl & F_TIMEOUT) throw Error{GMG_DEVICE_ERROR, "colouring did not terminate"};
    if (fl & F_OVERFLOW) throw Error{GMG_DEVICE_ERROR, "colouring: too many colours"};
    lv.ncolors = (int32_t)nco;
    tfree(s, wl);
    if (L.list) {
      tfree(s, L.list);
      tfree(s, L.mask);
      tfree(s, L.cnt);
    }
    tfree(s, ncol);
    return;
  }
  check_hip(hipMemsetAsync(ncol, 0, 4, s), "memset");
  int32_t* rounds = fresh_rounds(h);
  if (n <= kDrainItems) {
    k_color_drain<<<1, kDrainItems, 0, s>>>(lv.arp, lv.acol, n, key, lv.color, nullptr, nullptr, L, h.flags);
  } else {
    for (;;) {
      for (int t = 0; t < kColorBatch; ++t, ++k)
        k_color_round<<<grid, kBlock, 0, s>>>(lv.arp, lv.acol, n, key, lv.color, wl + ((k + 1) % 2) * n,
                                              wl + (k % 2) * n, rounds, k, L);
      int64_t left = 0;
      ScalarRead rd[1] = {{rounds + (k - 1), 4, &left}};
      read_scalars(h, rd, 1);
      if (left == 0) break;
      if (left <= kDrainItems) {
        k_color_drain<<<1, kDrainItems, 0, s>>>(lv.arp, lv.acol, n, key, lv.color, wl + ((k - 1) % 2) * n,
                                               rounds + (k - 1), L, h.flags);
        break;
      }
      if (k + kColorBatch > kMaxRounds) throw Error{GMG_DEVICE_ERROR, "colouring did not terminate"};
    }
  }
  {
    max_i32(lv.color, n, 1, ncol, s);
    int64_t nco = 0, fl = 0;
    ScalarRead rd[2] = {{ncol, 4, &nco}, {h.flags, 4, &fl}};
    read_scalars(h, rd, 2);
    if (fl & F_TIMEOUT) throw Error{GMG_DEVICE_ERROR, "colouring did not terminate"};
    lv.ncolors = (int32_t)nco;
  }
  // iterated-greedy passes: classes of the previous colouring from the highest
  // colour down (a pass never needs more colours, so the first count bounds
  // the classes of every pass)
  if (h.opt.color_passes > 0 && lv.ncolors > 1) {
    int32_t* other = (int32_t*)talloc(s, (size_t)n * 4);
    int32_t* cur = lv.color;
    int32_t* nxt = other;
    for (int p = 0; p < h.opt.color_passes; ++p) {
      fill_i32(nxt, -1, n, s);
      for (int32_t c = lv.ncolors - 1; c >= 0; --c)
        k_ig_class<<<grid, kBlock, 0, s>>>(lv.arp, lv.acol, n, cur, nxt, c);
      std::swap(cur, nxt);
    }
    check_hip(hipMemsetAsync(ncol, 0, 4, s), "memset");
    max_i32(cur, n, 1, ncol, s);
    if (cur != lv.color) check_hip(hipMemcpyAsync(lv.color, cur, (size_t)n * 4, hipMemcpyDeviceToDevice, s), "copy");
    int64_t nco = 0;
    ScalarRead rd[1] = {{ncol, 4, &nco}};
    read_scalars(h, rd, 1);
    lv.ncolors = (int32_t)nco;
    tfree(s, other);
  }
  tfree(s, wl);
  if (L.list) {
    tfree(s, L.list);
    tfree(s, L.mask);
    tfree(s, L.cnt);
  }
  tfree(s, ncol);
}

// ------------------------------------------------------------------ block order
// The grid of a level swept in block order (gmg_options.block_min_rows): the
// two coordinate axes of largest extent (the first smallest one dropped),
// cells of side w (1 + 2^-20), w the longest coupling of A_l along those axes.
// The host reads the extents and w, decides the grid, and the device assigns
// every point its brick (two cells of a row, shifted by one cell on odd rows)
// and its cell; block_colouring chooses between them.  The level keeps the
// colour order when it has no couplings or more than kMaxGridCells cells.
constexpr double kBlockMargin = 1.0 + 1.0 / (1 << 20);
constexpr int64_t kMaxGridCells = int64_t(1) << 22;

void block_order(Handle& h, Level& lv) {
  hipStream_t s = h.stream;
  const int64_t n = lv.n;
  unsigned long long* keys = (unsigned long long*)talloc(s, 9 * 8);
  k_grid_keys_init<<<1, kWave, 0, s>>>(keys);
  k_grid_extents<<<std::min(blocks_for(n), kReduceGrid), kBlock, 0, s>>>(lv.X, lv.arp, lv.acol, n, keys);
  int64_t kv[9];
  ScalarRead rd[9];
  for (int i = 0; i < 9; ++i) rd[i] = {keys + i, 8, &kv[i]};
  read_scalars(h, rd, 9);
  tfree(s, keys);
  auto from_key = [](int64_t k) {
    const uint64_t u = (uint64_t)k;
    const uint64_t b = (u >> 63) ? (u & ~(uint64_t(1) << 63)) : ~u;
    double d;
    std::memcpy(&d, &b, 8);
    return d;
  };
  double lo[3], ext[3], d[3];
  for (int a = 0; a < 3; ++a) {
    lo[a] = from_key(kv[a]);
    ext[a] = from_key(kv[3 + a]) - lo[a];
    std::memcpy(&d[a], &kv[6 + a], 8);
  }
  int drop = 0;
  for (int a = 1; a < 3; ++a)
    if (ext[a] < ext[drop]) drop = a;
  const int a0 = drop == 0 ? 1 : 0, a1 = drop == 2 ? 1 : 2;
  const double w = std::max(d[a0], d[a1]);
  if (!(w > 0.0)) return;
  const double side = w * kBlockMargin;
  const int64_t gx = (int64_t)std::floor(ext[a0] / side) + 1, gy = (int64_t)std::floor(ext[a1] / side) + 1;
  if (gx * gy > kMaxGridCells) return;
  lv.gx = (int32_t)gx;
  lv.gy = (int32_t)gy;
  lv.bcolor = (int32_t*)dalloc(h, (size_t)n * 4);
  lv.bcell = (int32_t*)talloc(s, (size_t)n * 4);
  lv.ccell = (int32_t*)talloc(s, (size_t)n * 4);
  k_grid_cells<<<blocks_for(n), kBlock, 0, s>>>(lv.X, n, a0, a1, lo[a0], lo[a1], side, lv.gx, lv.bcell, lv.ccell);
}

// The blocks and colouring of a level swept in block order: bricks of two
// cells, or single cells where a brick would hold more than kMaxBrickRows rows
// (lv.bcell receives the block of every row, lv.bcolor its colour), then
// DSATUR in every block (its rows numbered by ascending index).  Returns false,
// with the level's grid dropped, when a block has more than kMaxCellRows rows
// or needs kMaxCellColors colours; the level then takes the colour order.
bool block_colouring(Handle& h, Level& lv) {
  hipStream_t s = h.stream;
  const int64_t n = lv.n;
  // rows per brick and per cell: bricks are the blocks unless one of them
  // holds more than kMaxBrickRows rows
  const int64_t nbrick = (int64_t)(lv.gx / 2 + 1) * lv.gy, ncells = (int64_t)lv.gx * lv.gy;
  const int64_t cap = std::max(nbrick, ncells);
  int32_t* cnt = (int32_t*)talloc(s, (size_t)(cap + 1) * 4);
  int32_t* cnt2 = (int32_t*)talloc(s, (size_t)(ncells + 1) * 4);
  int32_t* slot = (int32_t*)talloc(s, (size_t)n * 4);
  int32_t* mx = (int32_t*)talloc(s, 4 * 4);
  fill_i32(cnt, 0, nbrick, s);
  fill_i32(cnt2, 0, ncells, s);
  fill_i32(mx, 0, 4, s);
  k_count_cells2<<<blocks_for(n), kBlock, 0, s>>>(lv.bcell, lv.ccell, n, cnt, cnt2);
  max_i32(cnt, nbrick, 0, mx, s);
  max_i32(cnt2, ncells, 0, mx + 3, s);
  int64_t mb = 0, mc = 0;
  {
    ScalarRead rd[2] = {{mx, 4, &mb}, {mx + 3, 4, &mc}};
    read_scalars(h, rd, 2);
  }
  tfree(s, cnt2);
  lv.bricks = mb <= kMaxBrickRows ? 1 : 0;
  const int64_t ncell = lv.bricks ? nbrick : ncells;
  const int64_t biggest = lv.bricks ? mb : mc;
  k_block_ids<<<blocks_for(n), kBlock, 0, s>>>(lv.bcell, lv.ccell, n, lv.gx, lv.bricks, lv.bcell, lv.bcolor);
  tfree(s, lv.ccell);
  lv.ccell = nullptr;
  fill_i32(cnt, 0, ncell + 1, s);
  k_cell_slots<<<blocks_for(n), kBlock, 0, s>>>(lv.bcell, n, cnt, slot);
  bool ok = biggest <= kMaxCellRows;
  if (ok) {
    int32_t* cptr = (int32_t*)talloc(s, (size_t)(ncell + 1) * 4);
    int32_t* rows = (int32_t*)talloc(s, (size_t)n * 4);
    scan_i32(cnt, cptr, ncell, s);
    k_cell_scatter<<<blocks_for(n), kBlock, 0, s>>>(lv.bcell, n, cptr, slot, rows);
    int32_t* deg = slot;                               // reused: in-cell degree of every row
    fill_i32(cnt, 0, ncell + 1, s);                    // reused: in-cell couplings of every cell
    k_incell_degree<<<blocks_for(n), kBlock, 0, s>>>(lv.arp, lv.acol, lv.bcell, n, deg, cnt);
    int32_t* cadj = (int32_t*)talloc(s, (size_t)(ncell + 1) * 4);
    scan_i32(cnt, cadj, ncell, s);
    int32_t* adj = (int32_t*)talloc(s, (size_t)std::max<int64_t>(lv.nnzA, 1) * 4);
    lv.color = (int32_t*)dalloc(h, (size_t)n * 4);
    k_cell_dsatur<<<(unsigned)ncell, kWave, 0, s>>>(cptr, rows, deg, cadj, lv.arp, lv.acol, lv.bcell, adj, lv.color,
                                                   mx + 1, mx + 2);
    int64_t top = 0, over = 0;
    ScalarRead rd[2] = {{mx + 1, 4, &top}, {mx + 2, 4, &over}};
    read_scalars(h, rd, 2);
    ok = over == 0;
    lv.ncolors = (int32_t)top + 1;
    tfree(s, cptr);
    tfree(s, rows);
    tfree(s, cadj);
    tfree(s, adj);
  }
  tfree(s, cnt);
  tfree(s, slot);
  tfree(s, mx);
  if (!ok) {                                           // the level takes the colour order
    tfree(s, lv.bcell);
    lv.bcell = nullptr;
    lv.bcolor = nullptr;
    lv.color = nullptr;
  }
  return ok;
}

namespace {

// The block sweep's layout of a level swept in block order (its solve
// numbering already sorted by (block colour, colour, index)).  The level keeps
// the launches per sweep class when a block does not fit the block kernel.
void block_layout(Handle& h, Level& lv, int32_t C) {
  hipStream_t s = h.stream;
  const int64_t n = lv.n;
  const int64_t ncell = lv.bricks ? (int64_t)(lv.gx / 2 + 1) * lv.gy : (int64_t)lv.gx * lv.gy;   // block ids
  const int64_t H = ncell;
  int32_t* cnt = (int32_t*)talloc(s, (size_t)ncell * 4);
  fill_i32(cnt, 0, ncell, s);
  k_count_cells<<<blocks_for(n), kBlock, 0, s>>>(lv.bcell, n, cnt);
  int32_t* flag = (int32_t*)talloc(s, (size_t)(4 * H + 1) * 4);
  int32_t* vid = (int32_t*)talloc(s, (size_t)(4 * H + 1) * 4);
  k_cell_flags<<<blocks_for(4 * H), kBlock, 0, s>>>(cnt, H, lv.gx, lv.bricks, flag);
  scan_i32(flag, vid, 4 * H, s);
  int64_t bs[5];
  {
    ScalarRead rd[5];
    for (int k = 0; k < 5; ++k) rd[k] = {vid + (int64_t)k * H, 4, &bs[k]};
    read_scalars(h, rd, 5);
  }
  const int32_t nblk = (int32_t)bs[4];
  tfree(s, cnt);
  tfree(s, flag);
  BlockView<double>& B = lv.view.B;
  B = BlockView<double>();
  if (nblk <= 0 || nblk > kMaxBlocks || C > kBlkMaxColors) {
    tfree(s, vid);
    return;
  }
  // rows of every block, ascending (a stable partition of the solve rows by block)
  int32_t* blk = (int32_t*)talloc(s, (size_t)n * 4);
  k_row_block<<<blocks_for(n), kBlock, 0, s>>>(lv.perm, lv.bcell, n, vid, H, lv.gx, lv.bricks, blk);
  tfree(s, vid);
  const int nb = blocks_for(n);
  int32_t* hist = (int32_t*)talloc(s, ((size_t)nblk * nb + 1) * 4);
  int32_t* hoffs = (int32_t*)talloc(s, ((size_t)nblk * nb + 1) * 4);
  int32_t* boff = (int32_t*)dalloc(h, (size_t)(nblk + 1) * 4);
  int32_t* brows = (int32_t*)dalloc(h, (size_t)n * 4);
  int32_t* bpos = (int32_t*)talloc(s, (size_t)n * 4);
  k_color_hist<<<nb, kBlock, (size_t)nblk * 4, s>>>(blk, n, nb, nblk, hist);
  scan_i32(hist, hoffs, (int64_t)nblk * nb, s);
  k_color_place<<<nb, kBlock, 0, s>>>(blk, n, nb, hoffs, nullptr, brows, bpos);
  k_color_ptr<<<blocks_for(nblk + 1), kBlock, 0, s>>>(hoffs, nb, nblk, 1, boff);
  tfree(s, hist);
  tfree(s, hoffs);
  // local row of every solve row; first local row of every colour
  int32_t* lpos = (int32_t*)talloc(s, (size_t)n * 4);
  k_local_rows<<<blocks_for(n), kBlock, 0, s>>>(bpos, blk, boff, n, lpos);
  tfree(s, bpos);
  int32_t* bcls = (int32_t*)dalloc(h, (size_t)nblk * (C + 1) * 4);
  k_block_cls<<<blocks_for((int64_t)nblk * (C + 1)), kBlock, 0, s>>>(boff, brows, lv.perm, lv.color, nblk, C, bcls);
  // halos (at most the blocks' entries each, compacted afterwards)
  int32_t* bad = (int32_t*)talloc(s, 4);
  fill_i32(bad, 0, 1, s);
  int32_t* cap = (int32_t*)talloc(s, (size_t)(nblk + 1) * 4);
  int32_t* tcap = (int32_t*)talloc(s, (size_t)(nblk + 1) * 4);
  int32_t* bw = (int32_t*)dalloc(h, (size_t)(nblk + 1) * 4);   // longest row of every block
  k_block_entries<<<blocks_for(nblk, kBlock / kWave), kBlock, 0, s>>>(lv.arp, lv.perm, brows, boff, nblk, cap, bw);
  scan_i32(cap, tcap, nblk, s);
  int32_t* tmp = (int32_t*)talloc(s, (size_t)std::max<int64_t>(lv.nnzA, 1) * 4);
  int32_t* hcnt = cap;                       // reused: distinct halo rows per block
  k_block_halo<<<nblk, kBlock, 0, s>>>(lv.arp, lv.acol, lv.perm, lv.iperm, blk, lv.bcolor, boff, brows, tmp, tcap,
                                       hcnt, bad);
  int32_t* hoff = (int32_t*)dalloc(h, (size_t)(nblk + 1) * 4);
  scan_i32(hcnt, hoff, nblk, s);
  int32_t* hlist = (int32_t*)dalloc(h, (size_t)std::max<int64_t>(lv.nnzA, 1) * 4);
  compact_long_segments(tmp, tcap, hoff, hlist, nblk, s);
  tfree(s, tmp);
  tfree(s, tcap);
  tfree(s, cap);
  // widths and the ELL offsets
  int32_t* sz = (int32_t*)talloc(s, (size_t)(nblk + 1) * 4);
  k_block_cells<<<blocks_for(nblk), kBlock, 0, s>>>(boff, bw, nblk, sz);
  int32_t* beoff = (int32_t*)dalloc(h, (size_t)(nblk + 1) * 4);
  scan_i32(sz, beoff, nblk, s);
  tfree(s, sz);
  int32_t* mx = (int32_t*)talloc(s, 5 * 4);
  fill_i32(mx, 0, 5, s);
  k_block_maxima<<<std::min(blocks_for(nblk), kReduceGrid), kBlock, 0, s>>>(boff, hoff, bw, nblk, C, mx);
  int64_t v[7] = {};
  {
    ScalarRead rd[7] = {{beoff + nblk, 4, &v[0]}, {mx, 4, &v[1]}, {mx + 1, 4, &v[2]}, {mx + 2, 4, &v[3]},
                        {bad, 4, &v[4]}, {mx + 3, 4, &v[5]}, {mx + 4, 4, &v[6]}};
    read_scalars(h, rd, 7);
  }
  tfree(s, mx);
  tfree(s, bad);
  const int64_t total = v[0], maxrows = v[1], maxhalo = v[2], maxw = v[3];
  const int64_t lds = (maxrows + maxhalo + 1) * 8;
  const bool fits = v[4] == 0 && maxrows <= 2 * kBlkThreads && maxw <= 64 && lds <= kBlkLdsMax &&
                    maxrows + maxhalo <= kBlkGather * kBlkThreads;
  if (fits) {
    int32_t* elx = (int32_t*)dalloc(h, (size_t)std::max<int64_t>(total, 1) * 4);
    double* elv = (double*)dalloc(h, (size_t)std::max<int64_t>(total, 1) * 8);
    k_block_ell<<<nblk, kBlock, 0, s>>>(lv.arp, lv.acol, lv.aval, lv.perm, lv.iperm, blk, lpos, boff, brows, hoff,
                                        hlist, bw, beoff, elx, elv);
    B.nblk = nblk;
    for (int k = 0; k < 5; ++k) B.bstart[k] = (int32_t)bs[k];
    B.ncls = C;
    B.rows_per_thread = maxrows <= kBlkThreads ? 1 : 2;
    B.width = maxw <= 32 ? 32 : 64;
    B.lds_bytes = (int32_t)lds;
    B.mlds[0] = (int32_t)v[5];
    B.mlds[1] = (int32_t)v[6];
    B.boff = boff;
    B.brows = brows;
    B.bcls = bcls;
    B.hoff = hoff;
    B.hlist = hlist;
    B.bw = bw;
    B.beoff = beoff;
    B.elx = elx;
    B.elv = elv;
    int32_t* rinfo = (int32_t*)dalloc(h, (size_t)n * 4);
    uint64_t* bmask = (uint64_t*)dalloc(h, (size_t)nblk * 8);
    k_block_rowinfo<<<blocks_for(n), kBlock, 0, s>>>(lv.arp, lv.perm, lv.color, brows, n, rinfo);
    k_block_mask<<<blocks_for(nblk), kBlock, 0, s>>>(bcls, nblk, C, bmask);
    B.rinfo = rinfo;
    B.bmask = bmask;
    // headers and gather lists (stride: the largest block plus the largest halo, in wavefronts)
    const int32_t gstride = (int32_t)((maxrows + maxhalo + kWave - 1) / kWave * kWave);
    BlockHdr* hdr = (BlockHdr*)dalloc(h, (size_t)nblk * sizeof(BlockHdr));
    int32_t* glist = (int32_t*)dalloc(h, (size_t)nblk * gstride * 4);
    k_block_gather<<<nblk, kBlock, 0, s>>>(boff, brows, hoff, hlist, bw, beoff, bmask, gstride, hdr, glist);
    B.hdr = hdr;
    B.glist = glist;
    B.gstride = gstride;
    lv.blk_entries = total;
  }
  tfree(s, blk);
  tfree(s, lpos);
}

}  // namespace

void block_values(Handle& h, Level& lv) {
  const BlockView<double>& B = lv.view.B;
  if (B.nblk == 0) return;
  k_block_values<<<B.nblk, kBlock, 0, h.stream>>>(lv.arp, lv.acol, lv.aval, lv.perm, B.boff, B.brows, B.bw, B.beoff,
                                                  B.nblk, (double*)B.elv);
}

namespace {

// CSR (source rows perm[r], columns through cmap) -> SELL-64 owned by the
// handle; *maxlen receives the longest row, *slots the allocated entry slots.
// uniform_nnz > 0 (the matrix's entries): every slice gets the width of the
// longest row when that stores at most kUniformSlack times the entries.
constexpr double kUniformSlack = 1.15;

// Coarse levels of at least this many rows also get P_l^T in original row order.
constexpr int64_t kRestrictOrigRows = 65536;

SellView make_sell(Handle& h, const int32_t* perm, const int32_t* cmap, const int32_t* rp, const int32_t* col,
                   const double* val, int64_t n, double* diag, int32_t* maxlen, int64_t* slots,
                   int64_t uniform_nnz = 0) {
  hipStream_t s = h.stream;
  const int64_t ns = (n + kSlice - 1) / kSlice;
  int32_t* len = (int32_t*)dalloc(h, (size_t)(n + 1) * 4);
  int32_t* ptr = (int32_t*)dalloc(h, (size_t)(ns + 1) * 4);
  int32_t* wsz = (int32_t*)talloc(s, (size_t)(ns + 1) * 4);
  int32_t* mx = (int32_t*)talloc(s, 4);
  check_hip(hipMemsetAsync(mx, 0, 4, s), "memset");
  k_row_len_width<<<blocks_for(ns * kSlice), kBlock, 0, s>>>(perm, rp, n, ns, len, wsz, mx);
  scan_i32(wsz, ptr, ns, s);
  int64_t tot = 0, ml = 0;
  ScalarRead rd[2] = {{ptr + ns, 4, &tot}, {mx, 4, &ml}};
  read_scalars(h, rd, 2);
  int32_t uw = 0;
  if (uniform_nnz > 0 && ml > 0 && (double)(ns * kSlice * ml) <= kUniformSlack * (double)uniform_nnz) {
    fill_i32(wsz, (int32_t)(ml * kSlice), ns, s);
    scan_i32(wsz, ptr, ns, s);
    tot = ns * kSlice * ml;
    uw = (int32_t)ml;
  }
  *maxlen = (int32_t)ml;
  *slots = tot + 1;
  int32_t* scol = (int32_t*)dalloc(h, (size_t)(tot + 1) * 4);
  double* sval = (double*)dalloc(h, (size_t)(tot + 1) * 8);
  if (ml <= kSliceFillMax) {
    const int pitch = (int)ml | 1;                 // odd: rows of the tile fall in different banks
    k_sell_fill_slice<<<(int)ns, kBlock, (size_t)kSlice * pitch * 12, s>>>(perm, cmap, rp, col, val, n, ptr, scol,
                                                                          sval, diag, pitch);
  } else {
    k_sell_fill<<<blocks_for(n), kBlock, 0, s>>>(perm, cmap, rp, col, val, n, ptr, scol, sval, diag);
  }
  tfree(s, wsz);
  tfree(s, mx);
  SellView v;
  v.ptr = ptr;
  v.col = scol;
  v.val = sval;
  v.len = len;
  v.uw = uw;
  return v;
}

// Lanes per row for the lane-parallel row kernels: each lane loads up to
// kLaneEntries entries of its row per pass.
int32_t lanes_for(int32_t maxlen) {
  int32_t r = 4;
  while (r < 64 && r * kLaneEntries < maxlen) r *= 2;
  return r;
}

}  // namespace

// An order of the finest points in which points near one another in the graph
// stand together, or null where the given order will do.  A row kernel gathers x
// at its rows' columns: with rows of one colour in an order without locality
// every gather of a wavefront is a cache line of its own.  The points are listed
// by the coarse point they belong to, the coarse points block by block, so that
// some 400 neighbours stand together, in ascending order within a coarse cell.
// Worth it only if the given order is not local: of consecutive points a quarter
// at most have their first couplings near one another (a mesh in grid order
// nearly all, points in random order nearly none).  Sweeps do not depend on the
// order within a colour.  1,000,000 points in random order, float: a colour 12.2 us,
// now 7.0; A p in double 112 us, now 51.  (In grid order, 1,048,576 points: 5.2 us a
// colour and 28 us, and nothing to gain.)
int32_t* cluster_order(Handle& h, const Level& lv, const Level& nx) {
  hipStream_t s = h.stream;
  const int64_t n = lv.n, nc = nx.n;
  if (nx.view.B.nblk <= 0 || !lv.label) return nullptr;
  int32_t* near = (int32_t*)talloc(s, 4);
  fill_i32(near, 0, 1, s);
  k_near_rows<<<std::min(blocks_for(n), kReduceGrid), kBlock, 0, s>>>(lv.arp, lv.acol, n, near);
  const int64_t m = read_i64(h, near, 4);
  tfree(s, near);
  if (4 * m >= n - 1) return nullptr;
  int32_t* order = (int32_t*)talloc(s, (size_t)n * 4);
  int32_t* pos = (int32_t*)talloc(s, (size_t)nc * 4);
  int32_t* slot = (int32_t*)talloc(s, (size_t)n * 4);
  int32_t* cnt = (int32_t*)talloc(s, (size_t)(nc + 1) * 4);
  int32_t* ptr = (int32_t*)talloc(s, (size_t)(nc + 1) * 4);
  k_block_pos<<<blocks_for(nc), kBlock, 0, s>>>(nx.view.B.brows, nx.perm, nc, pos);
  fill_i32(cnt, 0, nc + 1, s);
  k_cluster_count<<<blocks_for(n), kBlock, 0, s>>>(lv.label, pos, n, cnt, slot);
  scan_i32(cnt, ptr, nc, s);
  k_cluster_place<<<blocks_for(n), kBlock, 0, s>>>(lv.label, pos, ptr, slot, n, order);
  segment_sort_unique(order, ptr, cnt, nc, s);            // ascending in a cell, whatever the atomics' order
  tfree(s, pos);
  tfree(s, slot);
  tfree(s, cnt);
  tfree(s, ptr);
  return order;
}

void solve_layout(Handle& h, Level& lv, const Level* nx, const int32_t* t_rp, const int32_t* t_col,
                  const double* t_val) {
  hipStream_t s = h.stream;
  const int64_t n = lv.n;
  const int nb = blocks_for(n);
  const int C0 = lv.color ? lv.ncolors : 1;
  // sweep classes: the colours, or (block colour, colour) on a level swept in block order
  const int C = lv.bcolor ? 4 * C0 : C0;
  lv.perm = (int32_t*)dalloc(h, (size_t)n * 4);
  lv.iperm = (int32_t*)dalloc(h, (size_t)n * 4);
  int32_t* cptr = (int32_t*)dalloc(h, (size_t)(C + 1) * 4);
  int32_t *hist = nullptr, *off = nullptr;
  int32_t* stage = (int32_t*)pinned_staging((size_t)(2 * C + 1) * 4);
  if (lv.color) {
    // rows sorted by (sweep class, index); on levels swept by one workgroup by
    // (colour, width class, index)
    const int32_t* key = lv.color;
    int32_t* cls = nullptr;
    int K = 1;
    if (lv.bcolor) {
      cls = (int32_t*)talloc(s, (size_t)n * 4);
      k_sweep_class<<<blocks_for(n), kBlock, 0, s>>>(lv.bcolor, lv.color, n, C0, cls);
      key = cls;
    } else if (n <= kTailRows && (int64_t)C * kLenKeys * 4 <= 48 * 1024) {
      K = kLenKeys;
      cls = (int32_t*)talloc(s, (size_t)n * 4);
      k_len_class<<<blocks_for(n), kBlock, 0, s>>>(lv.color, lv.arp, n, cls);
      key = cls;
    }
    const int64_t classes = (int64_t)C * K;
    hist = (int32_t*)talloc(s, ((size_t)classes * nb + 1) * 4);
    off = (int32_t*)talloc(s, ((size_t)classes * nb + 1) * 4);
    int32_t* order = &lv == &h.L[0] && nx && n > kTailRows ? cluster_order(h, lv, *nx) : nullptr;
    if (order) {                              // (the finest level has neither of the keys above then)
      lv.clustered = true;
      cls = (int32_t*)talloc(s, (size_t)n * 4);
      k_gather_i32<<<blocks_for(n), kBlock, 0, s>>>(lv.color, order, n, cls);
      key = cls;
    }
    k_color_hist<<<nb, kBlock, (size_t)classes * 4, s>>>(key, n, nb, (int)classes, hist);
    scan_i32(hist, off, classes * nb, s);
    k_color_place<<<nb, kBlock, 0, s>>>(key, n, nb, off, order, lv.perm, lv.iperm);
    if (order) tfree(s, order);
    k_color_ptr<<<blocks_for(C + 1), kBlock, 0, s>>>(off, nb, C, K, cptr);
    if (cls) tfree(s, cls);
  } else {
    // the coarsest level keeps its numbering (it is solved directly)
    iota_i32(lv.perm, n, s);
    iota_i32(lv.iperm, n, s);
    stage[0] = 0;
    stage[1] = (int32_t)n;
    check_hip(hipMemcpyAsync(cptr, stage, 8, hipMemcpyHostToDevice, s), "copy");
  }
  lv.diag = (double*)dalloc(h, (size_t)n * 8);
  LevelView& v = lv.view;
  v.n = (int32_t)n;
  v.ncolors = C;
  v.cptr = cptr;
  v.A = make_sell(h, lv.perm, lv.iperm, lv.arp, lv.acol, lv.aval, n, lv.diag, &v.maxa, &lv.a_slots,
                  &lv == &h.L[0] ? lv.nnzA : 0);
  v.ra = lanes_for(v.maxa);
  v.diag = lv.diag;
  lv.x = (double*)dalloc(h, (size_t)n * 8);
  lv.b = (double*)dalloc(h, (size_t)n * 8);
  lv.r = (double*)dalloc(h, (size_t)n * 8);
  v.x = lv.x;
  v.b = lv.b;
  v.r = lv.r;
  if (lv.bcolor) {
    block_layout(h, lv, C0);
    tfree(s, lv.bcell);
    lv.bcell = nullptr;
  }
  // algorithmic bytes: 12 per entry (column + value), 28 per row (b, diagonal, row length, x write)
  lv.residual_bytes = 12.0 * (double)lv.nnzA + 28.0 * (double)n;
  int32_t* pre = nullptr;
  int32_t* cn = nullptr;
  if (lv.color) {
    pre = (int32_t*)talloc(s, (size_t)(n + 1) * 4);
    cn = (int32_t*)talloc(s, (size_t)C * 4);
    scan_i32(v.A.len, pre, n, s);
    k_color_nnz<<<blocks_for(C), kBlock, 0, s>>>(pre, cptr, C, cn);
  }
  if (nx) {
    // P: rows in this level's new numbering, columns in the next level's
    int32_t* qcol = (int32_t*)dalloc(h, (size_t)3 * n * 4);
    double* qval = (double*)dalloc(h, (size_t)3 * n * 8);
    int32_t* qcnt = (int32_t*)dalloc(h, (size_t)n * 4);
    k_p_layout<<<blocks_for(n), kBlock, 0, s>>>(lv.perm, nx->iperm, lv.pcol, lv.pval, lv.pcnt, n, qcol, qval,
                                                qcnt);
    v.q_col = qcol;
    v.q_val = qval;
    v.q_cnt = qcnt;
    // P^T: row I' = coarse row perm_c[I'], entries in ascending original fine index
    v.T = make_sell(h, nx->perm, lv.iperm, t_rp, t_col, t_val, nx->n, nullptr, &v.maxt, &lv.t_slots);
    if (nx->n >= kRestrictOrigRows) {
      int32_t mt = 0;
      v.To = make_sell(h, nullptr, lv.iperm, t_rp, t_col, t_val, nx->n, nullptr, &mt, &lv.to_slots);
      v.to_row = nx->iperm;
    }
    v.rt = lanes_for(v.maxt);
  }
  // colour ranges and per-colour entry counts (staging is reused by make_sell's reads, so copy last)
  stage = (int32_t*)pinned_staging((size_t)(2 * C + 1) * 4);
  check_hip(hipMemcpyAsync(stage, cptr, (size_t)(C + 1) * 4, hipMemcpyDeviceToHost, s), "copy");
  if (lv.color) check_hip(hipMemcpyAsync(stage + C + 1, cn, (size_t)C * 4, hipMemcpyDeviceToHost, s), "copy");
  sync(s, "solve layout");
  lv.color_ptr.assign(stage, stage + C + 1);
  lv.color_bytes.assign(C, 0.0);
  if (lv.color)
    for (int c = 0; c < C; ++c)
      lv.color_bytes[c] = 12.0 * (double)stage[C + 1 + c] + 28.0 * (double)(lv.color_ptr[c + 1] - lv.color_ptr[c]);
  tfree(s, pre);
  tfree(s, cn);
  tfree(s, hist);
  tfree(s, off);
}

// Slots per lane of the register form, with the depth of its load ring (as deep as
// 512 registers hold: a wavefront has a SIMD to itself up to 1024 columns).
template <int S>
void launch_inverse(const double* L, const double* U, int32_t n, double* inv, hipStream_t s) {
  constexpr int D = S <= 8 ? 8 : 4;
  k_coarse_inverse<S, D><<<n, kWave, 0, s>>>(L, U, n, inv);
}

void coarse_inverse(const double* L, const double* U, int64_t n64, double* inv, hipStream_t s) {
  const int32_t n = (int32_t)n64;
  switch ((n + kWave - 1) / kWave) {
    case 1: launch_inverse<1>(L, U, n, inv, s); break;
    case 2: launch_inverse<2>(L, U, n, inv, s); break;
    case 3: launch_inverse<3>(L, U, n, inv, s); break;
    case 4: launch_inverse<4>(L, U, n, inv, s); break;
    case 5: launch_inverse<5>(L, U, n, inv, s); break;
    case 6: launch_inverse<6>(L, U, n, inv, s); break;
    case 7: launch_inverse<7>(L, U, n, inv, s); break;
    case 8: launch_inverse<8>(L, U, n, inv, s); break;
    case 9: case 10: case 11: case 12: launch_inverse<12>(L, U, n, inv, s); break;
    case 13: case 14: case 15: case 16: launch_inverse<16>(L, U, n, inv, s); break;
    default:
      k_coarse_inverse_lds<<<n, kBlock, (size_t)n * 8, s>>>(L, U, n, inv);
  }
}

void coarse_factor(Handle& h, Level& lv) {
  hipStream_t s = h.stream;
  const int64_t n = lv.n;
  double* D = (double*)talloc(s, (size_t)n * n * 8);
  double* U = (double*)talloc(s, (size_t)n * n * 8);
  check_hip(hipMemsetAsync(D, 0, (size_t)n * n * 8, s), "memset");
  k_dense_scatter<<<blocks_for(n), kBlock, 0, s>>>(lv.arp, lv.acol, lv.aval, n, D);
  if (!h.chol) {                              // zeros above the diagonal
    h.chol = (double*)dalloc(h, (size_t)n * n * 8);
    check_hip(hipMemsetAsync(h.chol, 0, (size_t)n * n * 8, s), "memset");
  }
  if (!h.cinv) h.cinv = (double*)dalloc(h, (size_t)n * inv_ld(n) * 8);
  for (int64_t k0 = 0; k0 < n; k0 += kPanel) {
    const int64_t below = std::max<int64_t>(0, (n - k0 - 1) / kPanel);   // 32-row groups below the diagonal block
    const int64_t groups = std::max<int64_t>(1, below), tiles = k0 > 0 ? below * (below + 1) / 2 : 0;
    k_chol_step<<<(int)(groups + tiles), kCholT, 0, s>>>(D, (int32_t)n, (int32_t)k0, (int32_t)groups, h.chol, U, h.flags);
  }
  coarse_inverse(h.chol, U, n, h.cinv, s);
  h.ncoarse = n;
  check_flags(h, "coarsest factorisation");
  tfree(s, D);
  tfree(s, U);
}

// New values of A_l (same pattern) into its SELL layout and diagonal.
void refresh_values(Handle& h, Level& lv) {
  const LevelView& v = lv.view;
  k_sell_fill<<<blocks_for(lv.n), kBlock, 0, h.stream>>>(lv.perm, lv.iperm, lv.arp, lv.acol, lv.aval, lv.n, v.A.ptr,
                                                         (int32_t*)v.A.col, (double*)v.A.val, lv.diag);
}

template <class V>
void tail_layout(Handle& h, const Level& lv, TailRows<V>& R) {
  const LevelView& v = lv.view;
  if (!R.col) {
    tail_check();
    const int32_t W = std::min<int32_t>(tail_form(v.maxa), kTailWMax);
    R.nchunk = 0;
    for (size_t c = 0; c + 1 < lv.color_ptr.size(); ++c)
      R.nchunk += (lv.color_ptr[c + 1] - lv.color_ptr[c] + kWave - 1) / kWave;
    const size_t e = (size_t)R.nchunk * kWave * W;
    R.chunk = (int4*)dalloc(h, (size_t)R.nchunk * sizeof(int4));
    R.info = (int32_t*)dalloc(h, (size_t)lv.n * 4);
    R.col = (uint16_t*)dalloc(h, e * 2);
    R.val = (V*)dalloc(h, e * sizeof(V));
    if (tail_form(v.maxa) == kTailLong) {
      R.over = v.R.over;                       // the float copy: as the double one's
      R.oblocks = v.R.oblocks;
      if (!R.over) {
        int32_t* blocks = (int32_t*)talloc(h.stream, (size_t)R.nchunk * 4);
        int32_t* over = (int32_t*)dalloc(h, (size_t)(R.nchunk + 1) * 4);
        tail_over(v, R.nchunk, blocks, h.stream);
        scan_i32(blocks, over, R.nchunk, h.stream);
        R.oblocks = (int32_t)read_i64(h, over + R.nchunk, 4);
        R.over = over;
        tfree(h.stream, blocks);
      }
      R.ocol = (uint16_t*)dalloc(h, (size_t)R.oblocks * 16);
      R.oval = (V*)dalloc(h, (size_t)R.oblocks * 8 * sizeof(V));
    }
  }
  tail_fill<V>(v, R, h.stream);
}
template void tail_layout<double>(Handle&, const Level&, TailRows<double>&);
template void tail_layout<float>(Handle&, const Level&, TailRows<float>&);

}  // namespace gmg
