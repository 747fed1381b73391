// The V-cycle on levels with few rows (Alg. 2): all Gauss-Seidel sweeps of one
// level, the residual after them or the correction before them, in one
// workgroup; and the direct solve of the coarsest level, in the batched cycle
// with the restriction into it.  Grids of these kernels run one workgroup (or row of workgroups) per
// vector: one for the solve, kBatch for the batched forms, whose vectors are
// interleaved (entry (i, q) at i * stride + q).
#include <algorithm>

#include "rows.hpp"

namespace gmg {

namespace {

// One colour of such a level has 100-300 rows, so a kernel per colour is all
// launch latency (3 us against 0.3 us for its arithmetic), and the sweeps run
// in one workgroup with a barrier per colour.  A phase (colour) is a few
// wavefronts' worth of rows, each a chain of dependent operations on a nearly
// empty compute unit, so its time is the number of instructions a wavefront
// issues, and the latency of every load that was not issued phases ahead:
//  - each colour's rows (consecutive in the solve numbering) are cut into
//    chunks of one wavefront; chunk q belongs to wavefront q mod 8, which holds
//    its rows' entries in registers (up to W a row, the column a 16-bit byte
//    offset into the iterate in LDS), a row per lane.  A wavefront's control
//    flow is then its list of chunks: wait for the chunk's phase, sum, write;
//  - levels of at most 8 NB chunks are loaded once per call and stay; larger
//    ones reload a buffer as soon as its rows are done, NB chunks of the
//    wavefront (two to five phases each) ahead of their use;
//  - a wavefront loads 16 bytes per lane and instruction, contiguous, and only
//    as many entries as its chunk's longest row;
//  - on levels with rows of more than 32 entries (hubs, dense graphs) a form of
//    its own keeps one buffer and reads its rows' further entries in tiles of 16,
//    two of them in flight from before the barrier that opens the phase.
// Rows sum their terms in entry order; the diagonal entry points at a zero
// kept behind x in the sweeps (its product is +0, which leaves the sum
// unchanged: a sum that starts at +0 is never -0) and at the row itself in the
// residual.
__device__ __forceinline__ int32_t uniform(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }

// The row buffers load through buffer resources: a scalar base and bound, the
// thread's offset in one register and a uniform offset for the block of
// entries, so that no registers go to addresses.
using Rsrc = __amdgpu_buffer_rsrc_t;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ Rsrc make_rsrc(const void* p, int64_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)(uint32_t)bytes, 0x00020000);
}
__device__ __forceinline__ u32x4 bload16(Rsrc r, uint32_t voff, uint32_t soff) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, (int)voff, (int)soff, 0);
}

// A chunk's rows, one per lane: the loaded 16-byte blocks as they came (eight
// 16-bit column offsets, E values).
template <class V, int W>
struct TailBuf {
  static constexpr int E = 16 / sizeof(V);
  u32x4 c[W / 8];
  u32x4 v[W / E];
  V b, d;
  int32_t info;                            // the diagonal's entry
  int4 q;                                  // first row, rows, colour, entries of the longest row (all uniform)
};

// Value t of 16-byte blocks v.
template <class V>
__device__ __forceinline__ V tail_value(const u32x4* v, int t) {
  constexpr int E = 16 / sizeof(V);
  const u32x4 a = v[t / E];
  if constexpr (sizeof(V) == 8) {
    return __builtin_bit_cast(V, (uint64_t)a[2 * (t % E) + 1] << 32 | a[2 * (t % E)]);
  } else {
    const uint32_t u = a[t % E];           // a value of its own: bit_cast of a vector's element takes the first
    return __builtin_bit_cast(V, u);
  }
}

// Chunk `chunk`, whose entry of the chunk table is q.
template <class V, int W>
__device__ __forceinline__ void tail_load(const TailJob<V>& J, const V* b, int32_t chunk, int4 q, TailBuf<V, W>& f) {
  constexpr int E = TailBuf<V, W>::E;
  const uint32_t lane = threadIdx.x & (kWave - 1);
  f.q = int4{uniform(q.x), uniform(q.y), uniform(q.z), uniform(q.w)};
  const int32_t r = f.q.x + min((int32_t)lane, f.q.y - 1);
  f.b = b[(int64_t)r * J.stride];
  f.d = J.diag[r];
  f.info = J.A.info[r];
  constexpr uint32_t kC = W * 2 * kWave, kV = W * sizeof(V) * kWave;    // bytes of a chunk
  const Rsrc cr = make_rsrc(J.A.col, (int64_t)J.A.nchunk * kC), vr = make_rsrc(J.A.val, (int64_t)J.A.nchunk * kV);
#pragma unroll
  for (int g = 0; g < W / 8; ++g) {
    if (g == 0 || 8 * g < f.q.w) {
      f.c[g] = bload16(cr, lane * 16u, (uint32_t)chunk * kC + g * (kWave * 16u));
#pragma unroll
      for (int u = 0; u < 8 / E; ++u)
        f.v[8 / E * g + u] = bload16(vr, lane * 16u, (uint32_t)chunk * kV + (8 / E * g + u) * (kWave * 16u));
    }
  }
}

// The iterate's element at byte offset o: it starts the dynamic LDS, at LDS address 0
// as long as these kernels have no other (tail_check; an address of its own would cost
// an addition per gather).  A row's value is read by others only across a barrier, which
// orders these loads behind the stores through lds_raw.
template <class V>
__device__ __forceinline__ V lds_at(uint32_t o) {
  return *(const __attribute__((address_space(3))) V*)o;
}

// Two blocks of eight entries of the chunk's rows past their buffers.
template <class V>
struct TailTile {
  static constexpr int E = 16 / sizeof(V);
  u32x4 c[2], v[16 / E];
};

// Blocks g and g + 1 of the `blocks` past the buffers of the chunk in f, which begin
// at block `over` of the level's: a row's 16 bytes next to the next row's.  Past the
// last block the last again: the loads have no conditions, so that none waits for
// another.
template <class V, int W>
__device__ __forceinline__ void tail_tile(const TailJob<V>& J, const TailBuf<V, W>& f, int32_t over, int32_t blocks,
                                          int32_t g, TailTile<V>& t) {
  constexpr int E = TailTile<V>::E, B = 8 / E;
  const uint32_t lane = threadIdx.x & (kWave - 1), rows = (uint32_t)f.q.y, r = min(lane, rows - 1);
  const Rsrc cr = make_rsrc(J.A.ocol, (int64_t)J.A.oblocks * 16);
  const Rsrc vr = make_rsrc(J.A.oval, (int64_t)J.A.oblocks * (16 * B));
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const uint32_t at = (uint32_t)over + (uint32_t)min(g + h, blocks - 1) * rows;
    t.c[h] = bload16(cr, r * 16u, at * 16u);
#pragma unroll
    for (int u = 0; u < B; ++u) t.v[h * B + u] = bload16(vr, r * 16u, (at * B + u * rows) * 16u);
  }
}

// sum of the row's terms in entry order; Res: the diagonal's included.  The
// gathers of kTailGather entries are in flight together.
constexpr int kTailGather = 16;
template <bool Res, class V, int W>
__device__ __forceinline__ V tail_sum(const TailBuf<V, W>& f, int32_t row) {
  constexpr int G = W < kTailGather ? W : kTailGather;
  // the width and the columns are kept as they are: without this the compiler
  // computes every resident row's conditions and addresses once, outside the
  // sweeps, and spills them
  int32_t w = uniform(f.q.w);
  asm volatile("" : "+s"(w));
  const int32_t dp = f.info;
  V s = V(0);
#pragma unroll
  for (int g0 = 0; g0 < W; g0 += G) {
    if (g0 == 0 || g0 < w) {
      V xv[G];
#pragma unroll
      for (int h = 0; h < G; h += 8)
        if (g0 + h == 0 || g0 + h < w) {
          u32x4 c = f.c[(g0 + h) / 8];
          asm volatile("" : "+v"(c));
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            uint32_t o = (u & 1) ? c[u / 2] >> 16 : c[u / 2] & 0xFFFFu;
            if constexpr (Res) o = g0 + h + u == dp ? (uint32_t)row * (uint32_t)sizeof(V) : o;
            xv[h + u] = lds_at<V>(o);
          }
        }
#pragma unroll
      for (int h = 0; h < G; h += 8)
        if (g0 + h == 0 || g0 + h < w) {
#pragma unroll
          for (int u = 0; u < 8; ++u) s = s + tail_value<V>(f.v, g0 + h + u) * xv[h + u];
        }
    }
  }
  return s;
}

// The sum s of a chunk's rows taken on over the entries past their buffers, from the
// tiles a (blocks 0 and 1) and b (2 and 3), which it reads ahead of itself.  (Rows of
// 64 entries, 37 colours of 600 points: 1.8 us a phase.  Read from the SELL copy, each
// entry waiting for its column, these took 8.8, and four entries at a time in the
// kernel before that 4.1; 400 points of 106 couplings: 2.3, 17 and 5.6.)
template <bool Res, class V, int W>
__device__ __forceinline__ V tail_rest(const TailJob<V>& J, const TailBuf<V, W>& f, int32_t row, int32_t over,
                                       int32_t blocks, TailTile<V>& a, TailTile<V>& b, V s) {
  const int32_t dp = f.info - W;
  auto add = [&](const TailTile<V>& t, int32_t g) {
    V xv[16];
#pragma unroll
    for (int h = 0; h < 2; ++h)
      if (h == 0 || g + h < blocks) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          uint32_t o = (u & 1) ? t.c[h][u / 2] >> 16 : t.c[h][u / 2] & 0xFFFFu;
          if constexpr (Res) o = 8 * (g + h) + u == dp ? (uint32_t)row * (uint32_t)sizeof(V) : o;
          xv[8 * h + u] = lds_at<V>(o);
        }
      }
#pragma unroll
    for (int h = 0; h < 2; ++h)
      if (h == 0 || g + h < blocks) {
#pragma unroll
        for (int u = 0; u < 8; ++u) s = s + tail_value<V>(t.v, 8 * h + u) * xv[8 * h + u];
      }
  };
  int32_t g = 0;
  for (; g + 4 < blocks; g += 4) {
    add(a, g);
    tail_tile(J, f, over, blocks, g + 4, a);
    add(b, g + 2);
    tail_tile(J, f, over, blocks, g + 6, b);
  }
  add(a, g);
  if (g + 2 < blocks) add(b, g + 2);
  return s;
}

// LDS bytes of the iterate and its zero.
template <class V>
__host__ __device__ constexpr int32_t tail_lds(int32_t n) {
  return (int32_t)(((n + 1) * sizeof(V) + 15) & ~(size_t)15);
}

// nsweeps sweeps over the level's colours (descending if J.descending), the
// first J.skip colours of the first one already done; before them x += P x_c
// when J.q_col is set, after them r = b - A x when J.r is set.  vec: the
// vector's index in the interleaved arrays.  Phase p is colour p mod C of sweep
// p / C; the residual follows the last phase.
template <class V, int W, int NB, bool Stream, bool Long>
__device__ __forceinline__ void tail_run(const TailJob<V>& J, int32_t vec) {
  extern __shared__ double lds_raw[];
  V* xl = reinterpret_cast<V*>(lds_raw);                      // [n + 1]
  const int32_t t = threadIdx.x, lane = t & (kWave - 1), n = J.n, K = J.stride, C = J.ncolors;
  constexpr int kWaves = kTailT / kWave;
  const int32_t wv = uniform(t / kWave);
  const V* b = J.b + vec;
  V* x = J.x + vec;
  const bool desc = J.descending != 0;
  // this wavefront's chunks (wv, wv + 8, ..., or backwards from the last one
  // of its own), visited in the same order in every pass
  const int32_t mine = J.A.nchunk > wv ? (J.A.nchunk - wv + kWaves - 1) / kWaves : 0;
  const int32_t passes = J.nsweeps + (J.r ? 1 : 0);
  auto chunk_of = [&](int32_t k) { return wv + kWaves * (desc ? mine - 1 - k : k); };
  // visit i starts in buffer i; streaming, visits may run over several passes
  const int32_t visits = mine * passes;
  auto starts = [&](int i) { return Stream ? i < visits : i < mine; };
  auto start_chunk = [&](int i) { return chunk_of(Stream && i >= mine ? i % mine : i); };
  int4 q0[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) q0[i] = J.A.chunk[starts(i) ? start_chunk(i) : 0];
  if (t == 0) xl[n] = V(0);
  // the iterate, corrected from the coarser level: its vector first into LDS
  // (a gather of 64 cache lines takes the load path 64 cycles)
  constexpr int Q = kTailRows / kTailT;    // one round
  V* cl = reinterpret_cast<V*>(reinterpret_cast<char*>(lds_raw) + tail_lds<V>(n));    // [J.nc]; the chunk table follows in its place
  if (J.q_col) {
    const V* xc = J.xc + vec;
    for (int32_t i = t; i < J.nc; i += kTailT) cl[i] = xc[(int64_t)i * K];
  }
  {
    V xv[Q], p[Q][3];
    int32_t cnt[Q], j[Q][3];
#pragma unroll
    for (int u = 0; u < Q; ++u) {
      if (u * kTailT >= n) continue;
      const int32_t i = min(u * kTailT + t, n - 1);
      xv[u] = x[(int64_t)i * K];
      if (J.q_col) {
        cnt[u] = J.q_cnt[i];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          j[u][a] = J.q_col[(int64_t)a * n + i];
          p[u][a] = J.q_val[(int64_t)a * n + i];
        }
      }
    }
    if (J.q_col) {
      __syncthreads();
#pragma unroll
      for (int u = 0; u < Q; ++u) {
        if (u * kTailT >= n) continue;
        V acc = V(0);
#pragma unroll
        for (int a = 0; a < 3; ++a)
          if (a < cnt[u]) acc = acc + p[u][a] * cl[j[u][a]];
        xv[u] = xv[u] + acc;
      }
      __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < Q; ++u)
      if (u * kTailT + t < n) xl[u * kTailT + t] = xv[u];
  }
  TailBuf<V, W> buf[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i)
    if (starts(i)) tail_load<V, W>(J, b, start_chunk(i), q0[i], buf[i]);
  // the chunk table in LDS: a later load must not wait for memory to learn its width
  int4* ct = reinterpret_cast<int4*>(reinterpret_cast<char*>(lds_raw) + tail_lds<V>(n));
  int32_t* ot = reinterpret_cast<int32_t*>(ct + J.A.nchunk);  // Long: the chunks' first blocks past the buffers
  if constexpr (Stream)
    for (int32_t i = t; i < J.A.nchunk; i += kTailT) ct[i] = J.A.chunk[i];
  if constexpr (Long)
    if (J.A.over)                          // (a level of form kTailWMax in a group has none)
      for (int32_t i = t; i < J.A.nchunk; i += kTailT) ot[i] = J.A.over[i];
  __syncthreads();
  // phases done by the whole workgroup (one barrier ends each)
  int32_t phase = J.skip;
  auto reach = [&](int32_t p) {
    for (; phase < p; ++phase) __syncthreads();
  };
  // the phase of colour c in the sweep whose first phase is p0; the colour of the wavefront's chunk k
  auto phase_of = [&](int32_t c, int32_t p0) { return p0 + (desc ? C - 1 - c : c); };
  auto colour_of = [&](int32_t k) { return uniform(ct[chunk_of(k)].z); };
  // the chunk in f, the wavefront's k-th of the pass, in phase p: its rows swept, or
  // (Res) their residuals
  auto do_chunk = [&](auto res, const TailBuf<V, W>& f, int32_t k, int32_t p) {
    constexpr bool Res = decltype(res)::value;
    int32_t over = 0, blocks = 0;                             // past the buffers
    TailTile<V> ta, tb;
    if constexpr (Long) {
      blocks = (f.q.w - W) / 8;
      if (blocks > 0) {
        over = uniform(ot[chunk_of(k)]);
        tail_tile(J, f, over, blocks, 0, ta);
        tail_tile(J, f, over, blocks, 2, tb);
      }
    }
    reach(p);
    if (lane < f.q.y) {
      const int32_t row = f.q.x + lane;
      V s = tail_sum<Res>(f, row);
      if constexpr (Long)
        if (blocks > 0) s = tail_rest<Res>(J, f, row, over, blocks, ta, tb, s);
      if constexpr (Res) J.r[vec + (int64_t)row * K] = f.b - s;
      else xl[row] = (f.b - s) / f.d;
    }
  };
  auto sweep_chunk = [&](const TailBuf<V, W>& f, int32_t k, int32_t p) {
    if (p >= J.skip) do_chunk(std::integral_constant<bool, false>{}, f, k, p);
  };
  auto residual_chunk = [&](const TailBuf<V, W>& f, int32_t k, int32_t p) {
    do_chunk(std::integral_constant<bool, true>{}, f, k, p);
  };
  const int32_t end = J.nsweeps * C;
  if constexpr (Stream) {
    // k: place in the pass of the next visit; ahead: of the visit NB later
    int32_t k = 0, p0 = 0, left = visits, ahead = mine > 0 ? NB % mine : 0;
    while (left > 0) {
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        if (left > 0) {
          if (p0 < end) {
            const int32_t p = phase_of(uniform(buf[i].q.z), p0);
            sweep_chunk(buf[i], k, p);
            // end the phase before the reload when the wavefront's next chunk
            // is in a later one: the others need not wait for its loads to issue
            if (p >= J.skip && (left == 1 || k + 1 == mine || phase_of(NB > 1 ? uniform(buf[(i + 1) % NB].q.z) : colour_of(k + 1), p0) > p)) reach(p + 1);
          } else {
            residual_chunk(buf[i], k, end);
          }
          if (left > NB) tail_load<V, W>(J, b, chunk_of(ahead), ct[chunk_of(ahead)], buf[i]);
          ahead = ahead + 1 == mine ? 0 : ahead + 1;
          --left;
          if (++k == mine) {
            k = 0;
            p0 += C;
          }
        }
      }
    }
    reach(end);
  } else {
    for (int32_t p0 = 0; p0 < end; p0 += C) {
#pragma unroll
      for (int i = 0; i < NB; ++i)
        if (i < mine) sweep_chunk(buf[i], i, phase_of(uniform(buf[i].q.z), p0));
    }
    reach(end);
    if (J.r) {
#pragma unroll
      for (int i = 0; i < NB; ++i)
        if (i < mine) residual_chunk(buf[i], i, end);
    }
  }
  for (int32_t i = t; i < n; i += kTailT) x[(int64_t)i * K] = xl[i];
}

template <class V, int W, int NB, bool Stream, bool Long>
__global__ void __launch_bounds__(kTailT) k_tail(TailJob<V> J) {
  tail_run<V, W, NB, Stream, Long>(J, (int32_t)blockIdx.x);
}

// Grouped: job blockIdx.x / kBatch of the list, vector blockIdx.x % kBatch.
template <class V, int W, int NB, bool Stream, bool Long>
__global__ void __launch_bounds__(kTailT) k_gtail(const TailJob<V>* __restrict__ jobs,
                                                  const int32_t* __restrict__ members,
                                                  const int32_t* __restrict__ active) {
  const int32_t i = uniform((int32_t)blockIdx.x / kBatch);
  if (!active[members[i]]) return;
  const TailJob<V> J = jobs[i];
  tail_run<V, W, NB, Stream, Long>(J, (int32_t)blockIdx.x % kBatch);
}

// b_c = P^T r (or b_c given, when the job has no P^T) and x_c = A_c^-1 b_c in
// double: row i is the sum over k ascending of (A_c^-1 e_k)_i b_k.  A workgroup
// solves J.rows rows of one vector: in the batched cycle it restricts the whole
// vector itself while its columns of the inverse load (see kCoarseFused); it writes
// their products to LDS, and adds each row's products on one lane, two instructions
// a term.
constexpr int kCoarseAhead = 16;           // columns read from LDS ahead of their additions
constexpr int kCoarseM = 16;               // elements of the inverse a thread loads: coarse_rows(n) n / kTailT at most
constexpr int kCoarseStage = 8;            // elements of the residual a thread has in flight
constexpr int kCoarseChunk = 16;           // entries of a row of P^T whose loads are in flight together
// two wavefronts per SIMD: registers for those loads (left to itself the
// compiler keeps eight wavefronts and loads one entry after the other)
#define GMG_COARSE_BOUNDS __launch_bounds__(kTailT) __attribute__((amdgpu_waves_per_eu(2, 2)))
__host__ __device__ constexpr int32_t coarse_up(int32_t n) { return (n + kCoarseAhead - 1) / kCoarseAhead * kCoarseAhead; }

// acc and the `up` (a multiple of kCoarseAhead) products p, R apart, one after another.
template <int R>
__device__ __forceinline__ double coarse_add(double acc, const double* p, int32_t up) {
  const double* p0 = p;
  double q[2][kCoarseAhead];
#pragma unroll
  for (int u = 0; u < kCoarseAhead; ++u) q[0][u] = p[u * R];
  for (int32_t k = 0; k < up; k += 2 * kCoarseAhead) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      // the block after this one (past the end: the first again, not added)
      p = k + (h + 1) * kCoarseAhead < up ? p + kCoarseAhead * R : p0;
#pragma unroll
      for (int u = 0; u < kCoarseAhead; ++u) q[1 - h][u] = p[u * R];
      if (h == 0 || k + kCoarseAhead < up) {
#pragma unroll
        for (int u = 0; u < kCoarseAhead; ++u) acc = acc + q[h][u];
      }
    }
  }
  return acc;
}

template <class V, int R>
__device__ __forceinline__ void coarse_run(const CoarseJob<V>& J, int32_t group, int32_t vec) {
  extern __shared__ double lds_raw[];
  const int32_t n = J.n, K = J.stride, t = threadIdx.x;
  double* bc = lds_raw;                    // [n]
  const int32_t up = coarse_up(n);         // columns, rounded up
  double* m = lds_raw + up;                // [up][R]
  const int32_t i0 = group * R;
  const int64_t ld = inv_ld(n);
  const int32_t total = n * R;
  // all loads that need no other first: the columns of the inverse (at most
  // kCoarseM a thread, see coarse_rows) and the row's place in P^T
  double a[kCoarseM];
  const bool fused = J.T.ptr != nullptr;
  const int32_t ti = min(t, n - 1);
  SellRow row{};
  if (fused) row = sell_row(J.T, ti);
#pragma unroll
  for (int u = 0; u < kCoarseM; ++u) {
    if (u * kTailT >= total) continue;
    const int32_t e = min(u * kTailT + t, total - 1);
    a[u] = J.M[(int64_t)(e / R) * ld + min(i0 + (e & (R - 1)), n - 1)];
  }
  if (fused) {
    // the residual in LDS: a row gathers some 22 of its entries, each a cache line
    // of its own from memory
    const V* r = J.r + vec;
    V* rl = reinterpret_cast<V*>(m + up * R);
    for (int32_t e0 = 0; e0 < J.nf; e0 += kCoarseStage * kTailT) {
      V v[kCoarseStage];
#pragma unroll
      for (int u = 0; u < kCoarseStage; ++u)
        if (e0 + u * kTailT < J.nf) v[u] = r[(int64_t)min(e0 + u * kTailT + t, J.nf - 1) * K];
#pragma unroll
      for (int u = 0; u < kCoarseStage; ++u)
        if (e0 + u * kTailT + t < J.nf) rl[e0 + u * kTailT + t] = v[u];
    }
    __syncthreads();
    const auto* x = (const __attribute__((address_space(3))) V*)rl;
    for (int32_t i = t; i < n; i += kTailT) {
      if (i != t) row = sell_row(J.T, i);
      bc[i] = (double)row_sum_at<kCoarseChunk>(J.T, row, x, 1);
    }
  } else {
    for (int32_t i = t; i < n; i += kTailT) bc[i] = (double)J.b[vec + (int64_t)i * K];
  }
  __syncthreads();
  // the row's products, which one lane then only has to add; columns up to a
  // multiple of kCoarseAhead are zero (they leave a sum unchanged)
#pragma unroll
  for (int u = 0; u < kCoarseM; ++u) {
    const int32_t e = u * kTailT + t;
    if (e < total) m[e] = a[u] * bc[e / R];
  }
  if (total + t < up * R) m[total + t] = 0.0;
  __syncthreads();
  if (t < R && i0 + t < n) {
    const double acc = coarse_add<R>(0.0, m + t, up);
    J.x[vec + (int64_t)(i0 + t) * K] = (V)acc;
  }
}

template <class V, int R>
__global__ void GMG_COARSE_BOUNDS k_coarse(CoarseJob<V> J) {
  coarse_run<V, R>(J, (int32_t)blockIdx.x, (int32_t)blockIdx.y);
}

// Chunk q of a level whose colours begin at cptr[0 .. C]: its first row, rows, colour
// and the entries of its longest row, rounded up to a multiple of 8.
__device__ __forceinline__ int4 tail_chunk(const SellView& A, const int32_t* __restrict__ cptr, int32_t C, int32_t q) {
  const int lane = threadIdx.x & (kWave - 1);
  int32_t c = 0, before = 0, lo = 0, hi = 0;       // the colour that holds chunk q
  for (; c < C; ++c) {
    lo = cptr[c];
    hi = cptr[c + 1];
    const int32_t m = (hi - lo + kWave - 1) / kWave;
    if (q < before + m) break;
    before += m;
  }
  const int32_t r0 = lo + (q - before) * kWave, rows = min(hi - r0, kWave);
  int32_t w = lane < rows ? A.len[r0 + lane] : 0;
  for (int o = kWave / 2; o > 0; o >>= 1) w = max(w, __shfl_xor(w, o, kWave));
  return int4{r0, rows, c, (w + 7) & ~7};
}

__device__ __forceinline__ int32_t tail_chunk_index() {
  return uniform((int32_t)(blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave));
}

// The blocks of eight entries that every chunk's rows have past the first kTailWMax.
__global__ void __launch_bounds__(kBlock) k_tail_over(SellView A, const int32_t* __restrict__ cptr, int32_t C,
                                                      int32_t nchunk, int32_t* __restrict__ blocks) {
  const int32_t q = tail_chunk_index();
  if (q >= nchunk) return;
  const int4 k = tail_chunk(A, cptr, C, q);
  if ((threadIdx.x & (kWave - 1)) == 0) blocks[q] = max(0, (k.w - kTailWMax) / 8) * k.y;
}

// The same solve (b given) for coarsest levels of more than kCoarseAtOnce rows, of which
// a workgroup of coarse_run could take four at most with all their columns: kWideRows
// rows of a vector a workgroup, the columns in tiles of kWideCols, the next tile's loads
// in flight while one lane a row adds the products of one.  A direct solve of 1,100 rows
// takes 51 us in all, 2,000 61 and 4,032 84 (four or two rows a workgroup, a part of a
// cache line each: 59, 87 and 385; one lane a row from memory, 84, 125 and 212).
constexpr int kWideRows = 16, kWideCols = kCoarseM * kTailT / kWideRows;
template <class V>
__global__ void GMG_COARSE_BOUNDS k_coarse_wide(CoarseJob<V> J) {
  extern __shared__ double lds_raw[];
  constexpr int R = kWideRows;
  double* bc = lds_raw;                    // [kWideCols]
  double* m = lds_raw + kWideCols;         // [kWideCols][R]
  const int32_t n = J.n, K = J.stride, t = threadIdx.x, i0 = (int32_t)blockIdx.x * R, vec = (int32_t)blockIdx.y;
  const int64_t ld = inv_ld(n);
  double a[kCoarseM];
  V bv;
  auto load = [&](int32_t c0) {
#pragma unroll
    for (int u = 0; u < kCoarseM; ++u) {
      const int32_t e = u * kTailT + t;
      a[u] = J.M[(int64_t)min(c0 + e / R, n - 1) * ld + min(i0 + (e & (R - 1)), n - 1)];
    }
    bv = J.b[vec + (int64_t)min(c0 + t, n - 1) * K];
  };
  static_assert(kWideCols == kTailT, "a right-hand side per thread");
  load(0);
  double acc = 0.0;
  for (int32_t c0 = 0; c0 < n; c0 += kWideCols) {
    bc[t] = (double)bv;
    __syncthreads();                       // and the last tile's products are added
#pragma unroll
    for (int u = 0; u < kCoarseM; ++u) {
      const int32_t e = u * kTailT + t;
      m[e] = c0 + e / R < n ? a[u] * bc[e / R] : 0.0;
    }
    __syncthreads();
    load(min(c0 + kWideCols, n - 1));
    if (t < R) acc = coarse_add<R>(acc, m + t, coarse_up(min(kWideCols, n - c0)));
  }
  if (t < R && i0 + t < n) J.x[vec + (int64_t)(i0 + t) * K] = (V)acc;
}

// A_l (SELL, double) into the chunks' layout with values in V, a wavefront per
// chunk: its place in the colours, then a row per lane, padding with the zero
// behind the iterate and value 0.  The blocks past the buffers go round the grid's
// second dimension.
template <class V, int W>
__global__ void __launch_bounds__(kBlock) k_tail_fill(SellView A, const int32_t* __restrict__ cptr, int32_t C, int32_t n,
                                                      int32_t nchunk, int4* __restrict__ chunk,
                                                      int32_t* __restrict__ info, u32x4* __restrict__ col,
                                                      V* __restrict__ val, const int32_t* __restrict__ over,
                                                      u32x4* __restrict__ ocol, V* __restrict__ oval) {
  constexpr int E = 16 / sizeof(V);
  const int32_t q = tail_chunk_index();
  if (q >= nchunk) return;
  const int lane = threadIdx.x & (kWave - 1);
  const int4 k = tail_chunk(A, cptr, C, q);
  const int32_t rows = k.y, r = k.x + lane;
  const bool on = lane < rows;
  const int32_t len = on ? A.len[r] : 0;
  if (lane == 0 && blockIdx.y == 0) chunk[q] = k;
  const int64_t base = on ? A.ptr[r / kSlice] + (r & (kSlice - 1)) : 0;
  int32_t dp = -1;
  // entries e0 .. e0 + 7 of the row: a block of columns, 8 / E of values (v_at: the place of the h-th)
  auto block = [&](int32_t e0, u32x4& cols, auto v_at) {
    uint32_t o[8];
    V v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int32_t e = e0 + u;
      int32_t j = e < len ? A.col[base + (int64_t)e * kSlice] : n;
      v[u] = e < len ? (V)A.val[base + (int64_t)e * kSlice] : V(0);
      if (e < len && j == r) {
        dp = e;
        j = n;
      }
      o[u] = (uint32_t)j * (uint32_t)sizeof(V);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) cols[u] = o[2 * u] | o[2 * u + 1] << 16;
#pragma unroll
    for (int h = 0; h < 8 / E; ++h)
#pragma unroll
      for (int u = 0; u < E; ++u) v_at(h)[u] = v[h * E + u];
  };
#pragma unroll
  for (int e0 = 0; e0 < W; e0 += 8) {
    if (blockIdx.y > 0) break;
    u32x4 cw;
    block(e0, cw, [&](int h) { return val + (((int64_t)q * (W / E) + e0 / E + h) * kWave + lane) * E; });
    col[((int64_t)q * (W / 8) + e0 / 8) * kWave + lane] = cw;
  }
  if (over && on)
    for (int32_t g = (int32_t)blockIdx.y; W + 8 * g < k.w; g += (int32_t)gridDim.y) {
      const int64_t at = (int64_t)over[q] + (int64_t)g * rows;
      u32x4 cw;
      block(W + 8 * g, cw, [&](int h) { return oval + (at * (8 / E) + (int64_t)h * rows + lane) * E; });
      ocol[at + lane] = cw;
    }
  if (on && dp >= 0) info[r] = dp;
}

// Row buffers of a wavefront: what a thread's 256 registers take beside the
// gathered values.  A level whose chunks all have one stays resident; the
// streaming form has fewer, since a buffer being refilled needs registers twice.
template <class V, int W, bool Stream>
constexpr int tail_buffers() {
  if (sizeof(V) == 8) return W == 8 ? (Stream ? 4 : 7) : W == 16 ? (Stream ? 2 : 3) : 2;
  return W == 8 ? (Stream ? 4 : 8) : W == 16 ? (Stream ? 4 : 6) : (Stream ? 2 : 3);
}

// Calls f(W, NB, Stream, Long) as integral constants for levels of nchunk chunks
// (the most of a group) and the form of tail_form.
template <class V, class F>
void with_tail(int32_t form, int32_t nchunk, F&& f) {
  const std::integral_constant<bool, true> yes;
  const std::integral_constant<bool, false> no;
  auto go = [&](auto WC) {
    constexpr int w = decltype(WC)::value;
    const std::integral_constant<int, tail_buffers<V, w, false>()> resident;
    if (nchunk > resident.value * (kTailT / kWave))
      f(WC, std::integral_constant<int, tail_buffers<V, w, true>()>{}, yes, no);
    else
      f(WC, resident, no, no);
  };
  switch (form) {
    case 8: go(std::integral_constant<int, 8>{}); break;
    case 16: go(std::integral_constant<int, 16>{}); break;
    case kTailWMax: go(std::integral_constant<int, kTailWMax>{}); break;
    default:                               // one buffer beside the two tiles (two do not fit 256 registers in double)
      f(std::integral_constant<int, kTailWMax>{}, std::integral_constant<int, 1>{}, yes, yes);
  }
}

}  // namespace

int32_t tail_form(int32_t maxlen) { return maxlen <= 8 ? 8 : maxlen <= 16 ? 16 : maxlen <= kTailWMax ? kTailWMax : kTailLong; }

// Throws unless the dynamic LDS of every one-workgroup kernel starts at address 0 (lds_at).
void tail_check() {
  static const bool checked = [] {
    auto at_zero = [](const void* kernel) {
      hipFuncAttributes a;
      check_hip(hipFuncGetAttributes(&a, kernel), "attributes of the one-workgroup kernels");
      if (a.sharedSizeBytes != 0) throw Error{GMG_DEVICE_ERROR, "one-workgroup kernel with static LDS"};
    };
    auto all = [&](auto zero) {
      using V = decltype(zero);
      for (int32_t form : {8, 16, kTailWMax, kTailLong})
        for (int32_t nchunk : {1, (int32_t)kTailRows})         // resident and streamed
          with_tail<V>(form, nchunk, [&](auto WC, auto BC, auto SC, auto LC) {
            constexpr int W = decltype(WC)::value, NB = decltype(BC)::value;
            constexpr bool Stream = decltype(SC)::value, Long = decltype(LC)::value;
            at_zero((const void*)k_tail<V, W, NB, Stream, Long>);
            at_zero((const void*)k_gtail<V, W, NB, Stream, Long>);
          });
    };
    all(0.0);
    all(0.0f);
    return true;
  }();
  (void)checked;
}

template <class V>
size_t tail_lds_bytes(const TailRows<V>& A, int32_t n, int32_t nc) {
  return (size_t)tail_lds<V>(n) + std::max((size_t)A.nchunk * (sizeof(int4) + (A.over ? 4 : 0)), (size_t)nc * sizeof(V));
}

template <class V>
TailJob<V> tail_job(const LevelViewT<V>& v, int32_t stride) {
  TailJob<V> J;
  J.n = v.n;
  J.ncolors = v.ncolors;
  J.stride = stride;
  J.maxlen = v.maxa;
  J.A = v.R;
  J.diag = v.diag;
  J.b = v.b;
  J.x = v.x;
  return J;
}

template <class V>
TailJob<V> tail_pre_job(const LevelViewT<V>& v, int32_t stride, int32_t nu, int32_t skip) {
  TailJob<V> J = tail_job(v, stride);
  J.nsweeps = nu;
  J.skip = nu > 0 ? skip : 0;
  J.r = v.r;
  return J;
}

template <class V>
TailJob<V> tail_post_job(const LevelViewT<V>& v, const LevelViewT<V>& c, int32_t stride, int32_t nu,
                         bool descending) {
  TailJob<V> J = tail_job(v, stride);
  J.nsweeps = nu;
  J.descending = descending ? 1 : 0;
  J.q_col = v.q_col;
  J.q_val = v.q_val;
  J.q_cnt = v.q_cnt;
  J.xc = c.x;
  J.nc = c.n;
  return J;
}

template <class V>
void tail_sweeps(const TailJob<V>& J, int32_t form, int32_t vectors, hipStream_t s) {
  if (!J.A.col || form != tail_form(J.maxlen) || J.n > kTailRows)
    throw Error{GMG_DEVICE_ERROR, "tail level without its row layout"};
  with_tail<V>(form, J.A.nchunk, [&](auto WC, auto BC, auto SC, auto LC) {
    k_tail<V, decltype(WC)::value, decltype(BC)::value, decltype(SC)::value, decltype(LC)::value>
        <<<vectors, kTailT, tail_lds_bytes(J.A, J.n, J.nc), s>>>(J);
  });
}

template <class V>
void gtail_sweeps(const TailJob<V>* jobs, const int32_t* members, int32_t count, int32_t form, int32_t nchunk, size_t lds,
                  const int32_t* active, hipStream_t s) {
  if (count <= 0) return;
  with_tail<V>(form, nchunk, [&](auto WC, auto BC, auto SC, auto LC) {
    k_gtail<V, decltype(WC)::value, decltype(BC)::value, decltype(SC)::value, decltype(LC)::value>
        <<<count * kBatch, kTailT, lds, s>>>(jobs, members, active);
  });
}

// Rows a workgroup of the coarsest solve of up to kCoarseAtOnce takes: kCoarseM elements
// of the inverse a thread, at most 64 KiB in LDS.  More rows per workgroup mean fewer
// copies of the restriction, fewer mean more load paths.
int32_t coarse_rows(int64_t n) { return n <= 512 ? 16 : 8; }
template <class V>
size_t coarse_lds(const CoarseJob<V>& J) {
  return (size_t)coarse_up(J.n) * 8 * (1 + J.rows) + (J.T.ptr ? (size_t)J.nf * sizeof(V) : 0);
}

template <class F>
void with_rows(int32_t R, F&& f) {
  switch (R) {
    case 16: f(std::integral_constant<int, 16>{}); break;
    default: f(std::integral_constant<int, 8>{}); break;
  }
}

template <class V>
void coarse_solve(const CoarseJob<V>& J, int32_t vectors, hipStream_t s) {
  if (J.T.ptr && (J.n > kCoarseAtOnce || (int64_t)J.nf * (int64_t)sizeof(V) > kCoarseStaged))
    throw Error{GMG_DEVICE_ERROR, "level too large to restrict in the coarsest solve"};
  if (J.n > kCoarseAtOnce) {
    k_coarse_wide<V><<<dim3((J.n + kWideRows - 1) / kWideRows, vectors), kTailT,
                       (size_t)kWideCols * (1 + kWideRows) * 8, s>>>(J);
    return;
  }
  with_rows(J.rows, [&](auto RC) {
    k_coarse<V, decltype(RC)::value><<<dim3((J.n + J.rows - 1) / J.rows, vectors), kTailT, coarse_lds(J), s>>>(J);
  });
}

void tail_over(const LevelView& v, int32_t nchunk, int32_t* blocks, hipStream_t s) {
  k_tail_over<<<blocks_for(nchunk, kBlock / kWave), kBlock, 0, s>>>(v.A, v.cptr, v.ncolors, nchunk, blocks);
}

template <class V>
void tail_fill(const LevelView& v, const TailRows<V>& R, hipStream_t s) {
  auto go = [&](auto WC) {
    k_tail_fill<V, decltype(WC)::value><<<dim3(blocks_for(R.nchunk, kBlock / kWave), R.over ? 16 : 1), kBlock, 0, s>>>(
        v.A, v.cptr, v.ncolors, v.n, R.nchunk, (int4*)R.chunk, (int32_t*)R.info, (u32x4*)R.col, (V*)R.val, R.over,
        (u32x4*)R.ocol, (V*)R.oval);
  };
  switch (tail_form(v.maxa)) {
    case 8: go(std::integral_constant<int, 8>{}); break;
    case 16: go(std::integral_constant<int, 16>{}); break;
    default: go(std::integral_constant<int, kTailWMax>{}); break;
  }
}

#define GMG_INSTANTIATE_TAIL(V)                                                                                 \
  template size_t tail_lds_bytes<V>(const TailRows<V>&, int32_t, int32_t);                                                               \
  template TailJob<V> tail_pre_job<V>(const LevelViewT<V>&, int32_t, int32_t, int32_t);                        \
  template TailJob<V> tail_post_job<V>(const LevelViewT<V>&, const LevelViewT<V>&, int32_t, int32_t, bool);    \
  template void tail_sweeps<V>(const TailJob<V>&, int32_t, int32_t, hipStream_t);                              \
  template void gtail_sweeps<V>(const TailJob<V>*, const int32_t*, int32_t, int32_t, int32_t, size_t, const int32_t*,   \
                                hipStream_t);                                                                  \
  template void coarse_solve<V>(const CoarseJob<V>&, int32_t, hipStream_t);                                     \
  template void tail_fill<V>(const LevelView&, const TailRows<V>&, hipStream_t);
GMG_INSTANTIATE_TAIL(double)
GMG_INSTANTIATE_TAIL(float)
#undef GMG_INSTANTIATE_TAIL

}  // namespace gmg
