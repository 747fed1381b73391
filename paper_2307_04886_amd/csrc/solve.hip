// V-cycle kernels (Alg. 2): multicolour Gauss-Seidel, residual, restriction
// by P^T, prolongation and correction, norms.
//
// Every kernel is written once for the value type V of the level data: double
// for the solve of Alg. 1, float for the mixed-precision CG preconditioner.
// The levels with few rows and the coarsest solve are in tail.hip.
#include <type_traits>

#include "rows.hpp"

namespace gmg {

namespace {


template <class V>
__device__ __forceinline__ void prolong_row(const LevelViewT<V>& L, const V* __restrict__ xc, V* x, int32_t i) {
  const int32_t c = L.q_cnt[i];
  V acc = V(0);
  V v[3], u[3];
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    v[t] = L.q_val[(int64_t)t * L.n + i];
    u[t] = xc[L.q_col[(int64_t)t * L.n + i]];
  }
#pragma unroll
  for (int t = 0; t < 3; ++t)
    if (t < c) acc = acc + v[t] * u[t];
  x[i] = x[i] + acc;
}

// Level 0's one-lane row sum: per-slice widths (row lengths read), or the
// uniform slice width (U) when the level's SELL has one.
template <int CH, bool U, class V>
__device__ __forceinline__ V row_sum_fine(const Sell<V>& A, int32_t r, const V* x, int32_t skip) {
  if constexpr (U) return row_sum_uni<CH>(A, r, x, skip);
  else return row_sum_seq<CH>(A, r, x, skip);
}

// One colour of a Gauss-Seidel sweep on level 0, rows [r0, r1):
//   x_r <- (b_r - sum_{j != r} A_rj x_j) / A_rr.
// Rows of one colour are not coupled, so they update in parallel.
template <int CH, bool U, class V>
__global__ void __launch_bounds__(kBlock) k_gs_color_fine(Sell<V> A, const V* __restrict__ diag,
                                                          const V* __restrict__ b, V* x, int32_t r0, int32_t r1) {
  const int32_t r = (r0 & ~(kSlice - 1)) + (int32_t)(xcd_block() * kBlock + threadIdx.x);
  if (r < r0 || r >= r1) return;
  const V br = b[r], dr = diag[r];        // issued with the row's loads
  const V acc = row_sum_fine<CH, U>(A, r, x, r);
  x[r] = (br - acc) / dr;
}

// The same update on a Galerkin level, R lanes per row.
template <int R, class V>
__global__ void __launch_bounds__(kBlock) k_gs_color(Sell<V> A, const V* __restrict__ diag,
                                                     const V* __restrict__ b, V* x, int32_t r0, int32_t r1,
                                                     int32_t maxlen) {
  const int64_t g = ((int64_t)xcd_block() * kBlock + threadIdx.x) / R;
  const int32_t r = r0 + (int32_t)g;
  const bool active = r < r1;
  const int32_t rc = active ? r : r0;     // in range for every lane: the loads need no branch
  const V br = b[rc], dr = diag[rc];
  const V acc = row_sumR<R>(A, r, active, x, r, maxlen);
  if (active && (threadIdx.x & (R - 1)) == 0) x[r] = (br - acc) / dr;
}

// One block colour of a Gauss-Seidel sweep in block order (levels swept by
// blocks): one workgroup per block (grid cell) of that colour.  Rows of one
// block colour in different blocks are never coupled, so the blocks run at
// once; inside a block the colours run one after the other, separated by
// workgroup barriers, with the block's iterates and the values of its halo
// (the rows of other blocks its rows read, which this launch does not change)
// in LDS.  Thread p holds local rows p and p + kBlkThreads (R of them) with
// their entries in registers: the LDS slot of each column and its value, in
// the row's entry order, the diagonal replaced by a zero term (slot `pad`
// holds +0), so x_i <- (b_i - sum_{j != i} A_ij x_j) / A_ii is computed with
// the terms added in entry order, as on the other paths.  NG gather slots per
// thread cover the gather list (NG * kBlkThreads >= its stride); they are
// read branch-free (slots past the stride re-read its last entry), so the
// list's loads are in flight together.  The register budget sets how many
// workgroups a compute unit holds at once (at 168 VGPRs, three: 768 on the
// chip), and so whether a level's blocks of one colour run in a single round;
// a variant that needs more registers must be measured for it.
template <int R, int K, int NG, class V>
__global__ void __launch_bounds__(kBlkThreads) k_gs_block(BlockView<V> B, const V* __restrict__ bvec,
                                                          const V* __restrict__ diag, V* x, int32_t blk0,
                                                          int32_t c_begin, int32_t descending) {
  extern __shared__ double lds_raw[];
  V* xl = reinterpret_cast<V*>(lds_raw);
  const int32_t b = blk0 + (int32_t)blockIdx.x;
  // first: the header and the gather list (addresses from the block index
  // alone), then the entries, row data and iterates they point to
  const BlockHdr hd = B.hdr[b];
  const int32_t* gl = B.glist + (int64_t)b * B.gstride;
  int32_t gi[NG];
#pragma unroll
  for (int j = 0; j < NG; ++j) gi[j] = gl[min((int32_t)threadIdx.x + j * kBlkThreads, B.gstride - 1)];
  const int32_t r0 = hd.r0, rows = hd.rows, nh = hd.nh, w = hd.w, e0 = hd.e0;
  const int C = B.ncls;
  const int32_t pad = rows + nh;
  const uint64_t present = hd.mask;          // colours with rows in the block
  // Row data and entries.  Two forms with the same values in every slot that
  // is used.  Double: per-lane conditional loads (lanes past the block's rows
  // and slots past its width take the zero term), which fit 168 VGPRs.  Float:
  // no branch inside a wavefront (with per-lane conditions the compiler waited
  // for each load before issuing the next): a wavefront without rows of the
  // block skips them (its registers are never read), lanes past the block's
  // rows re-read its last row (masked where the rows are swept) and slots
  // past the width re-read its last slot (their products are replaced by zero
  // where the row is summed).
  constexpr bool kClamp = sizeof(V) == 4;
  const int32_t wbase = __builtin_amdgcn_readfirstlane((int32_t)threadIdx.x & ~(kWave - 1));
  int32_t info[R];
  V bv[R], dv[R];
  int32_t lx[R][K];
  V lv[R][K];
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const int32_t p = (int32_t)threadIdx.x + q * kBlkThreads;
    if constexpr (kClamp) {
      const int32_t pc = min(p, rows - 1);
      if (wbase + q * kBlkThreads < rows) {
        info[q] = B.rinfo[r0 + pc];
#pragma unroll
        for (int t = 0; t < K; ++t) {
          const int32_t o = e0 + min(t, w - 1) * rows + pc;
          lx[q][t] = B.elx[o];
          lv[q][t] = B.elv[o];
        }
      }
    } else {
      const bool own = p < rows;
      info[q] = own ? B.rinfo[r0 + p] : 0;
#pragma unroll
      for (int t = 0; t < K; ++t) {
        const bool e = own && t < w;
        lx[q][t] = e ? B.elx[e0 + t * rows + p] : pad;
        lv[q][t] = e ? B.elv[e0 + t * rows + p] : V(0);
      }
    }
  }
  // the block's own rows (thread p holds rows p, p + kBlkThreads, ...) and its halo
#pragma unroll
  for (int j = 0; j < NG; ++j) {
    const int32_t k = (int32_t)threadIdx.x + j * kBlkThreads;
    if (k < pad) {
      xl[k] = x[gi[j]];
      if (j < R && k < rows) {
        bv[j] = bvec[gi[j]];
        dv[j] = diag[gi[j]];
      }
    }
  }
  if (threadIdx.x == 0) xl[pad] = V(0);
  __syncthreads();
  for (int kk = c_begin; kk < C; ++kk) {
    const int c = descending ? C - 1 - kk : kk;
    if (!((present >> c) & 1)) continue;                // no row of this colour in the block
#pragma unroll
    for (int q = 0; q < R; ++q) {
      if ((int32_t)threadIdx.x + q * kBlkThreads < rows && (info[q] & 0xFF) == c) {
        const int32_t len = info[q] >> 8;
        // every gather of the row is issued at once, then the products are
        // added in entry order, in chunks of 8 up to the row's length
        // (terms past the row are +0); the largest shape works a chunk at a
        // time, within its registers
        constexpr int G = R * K <= 64 ? K : 8;
        V s = V(0);
#pragma unroll
        for (int g0 = 0; g0 < K; g0 += G) {
          if (g0 < w) {
            V pr[G];
#pragma unroll
            for (int t = 0; t < G; ++t)
              pr[t] = (!kClamp || g0 + t < w ? lv[q][g0 + t] : V(0)) * xl[lx[q][g0 + t]];
#pragma unroll
            for (int t0 = 0; t0 < G; t0 += 8) {
              if (g0 + t0 < len) {
#pragma unroll
                for (int u = 0; u < 8; ++u) s = s + pr[t0 + u];
              }
            }
          }
        }
        xl[(int32_t)threadIdx.x + q * kBlkThreads] = (bv[q] - s) / dv[q];
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const int32_t p = (int32_t)threadIdx.x + q * kBlkThreads;
    if (p < rows) x[gi[q]] = xl[p];
  }
}

// r = b - A x on level 0
template <int CH, bool U, class V>
__global__ void __launch_bounds__(kBlock) k_residual_fine(Sell<V> A, const V* __restrict__ b,
                                                          const V* __restrict__ x, V* __restrict__ res,
                                                          int64_t n) {
  const int64_t r = (int64_t)xcd_block() * kBlock + threadIdx.x;
  if (r >= n) return;
  res[r] = b[r] - row_sum_fine<CH, U>(A, (int32_t)r, x, -1);
}

// r = b - A x on a Galerkin level, R lanes per row
template <int R, class V>
__global__ void __launch_bounds__(kBlock) k_residual(Sell<V> A, const V* __restrict__ b, const V* __restrict__ x,
                                                     V* __restrict__ res, int64_t n, int32_t maxlen) {
  const int64_t g = ((int64_t)xcd_block() * kBlock + threadIdx.x) / R;
  const bool active = g < n;
  const V acc = row_sumR<R>(A, (int32_t)g, active, x, -1, maxlen);
  if (active && (threadIdx.x & (R - 1)) == 0) res[g] = b[g] - acc;
}

// r = b - A x on level 0 (double), plus per-block partial sums of r^2 (fixed
// grid: deterministic).
template <int CH, bool U>
__global__ void __launch_bounds__(kBlock) k_residual_norm(SellView A, const double* __restrict__ b,
                                                          const double* __restrict__ x,
                                                          double* __restrict__ res, int64_t n,
                                                          double* partials) {
  // logical block lb covers rows lb * kBlock + k * gridDim.x * kBlock and
  // writes partials[lb], whichever XCD runs it
  const uint32_t lb = xcd_block();
  double sq = 0.0;
  for (int64_t r = (int64_t)lb * kBlock + threadIdx.x; r < n; r += (int64_t)gridDim.x * kBlock) {
    const double v = b[r] - row_sum_fine<CH, U>(A, (int32_t)r, x, -1);
    res[r] = v;
    sq += v * v;
  }
  double t = block_sum(sq);
  if (threadIdx.x == 0) partials[lb] = t;
}

__global__ void __launch_bounds__(kBlock) k_norm_partials(const double* v, int64_t n, double* partials) {
  double sq = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBlock)
    sq += v[i] * v[i];
  double t = block_sum(sq);
  if (threadIdx.x == 0) partials[blockIdx.x] = t;
}

// The norm into out and, when host_out is set (pinned host memory), there too,
// so that the host sees it without a copy.
__global__ void __launch_bounds__(kBlock) k_finish_norm(const double* partials, double* out, double* host_out) {
  double s = 0.0;
  for (int i = threadIdx.x; i < kNormBlocks; i += kBlock) s += partials[i];
  double t = block_sum(s);
  if (threadIdx.x == 0) {
    const double v = sqrt(t);
    *out = v;
    if (host_out)
      __hip_atomic_store(reinterpret_cast<uint64_t*>(host_out), __builtin_bit_cast(uint64_t, v), __ATOMIC_RELEASE,
                         __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

// b_c[I] = sum over row I of P^T (ascending original fine index) of P[i,I] r_i,
// and the coarse iterate starts from zero: x_c[I] = 0.  Rows I < first (the
// first colour of the coarse level, when its first pre-smoothing colour is
// folded in here) take that colour's Gauss-Seidel update from the zero
// iterate instead: every neighbour term is a product with +0, the sum is +0,
// and x_c[I] = (b_c[I] - 0) / A_c[I,I], the value the sweep would write.
template <int R, class V>
__global__ void __launch_bounds__(kBlock) k_restrict(Sell<V> T, const V* __restrict__ r, V* __restrict__ bc,
                                                     V* __restrict__ xc, int64_t nc, int32_t maxlen,
                                                     const V* __restrict__ diag_c, int32_t first,
                                                     const int32_t* __restrict__ orow) {
  const int64_t g = ((int64_t)xcd_block() * kBlock + threadIdx.x) / R;
  const bool active = g < nc;
  const V acc = row_sumR<R>(T, (int32_t)g, active, r, -1, maxlen);
  if (active && (threadIdx.x & (R - 1)) == 0) {
    const int64_t o = orow ? orow[g] : g;        // T's row g is coarse row o
    bc[o] = acc;
    xc[o] = o < first ? (acc - V(0)) / diag_c[o] : V(0);
  }
}

// The same restriction with one lane per coarse row (its terms loaded CH at a
// time and added in entry order, as by the R-lane form).
template <int CH, class V>
__global__ void __launch_bounds__(kBlock) k_restrict_seq(Sell<V> T, const V* __restrict__ r, V* __restrict__ bc,
                                                         V* __restrict__ xc, int64_t nc,
                                                         const V* __restrict__ diag_c, int32_t first,
                                                         const int32_t* __restrict__ orow) {
  const int64_t g = (int64_t)xcd_block() * kBlock + threadIdx.x;
  if (g >= nc) return;
  const V acc = row_sum_seq<CH>(T, (int32_t)g, r, -1);
  const int64_t o = orow ? orow[g] : g;          // T's row g is coarse row o
  bc[o] = acc;
  xc[o] = o < first ? (acc - V(0)) / diag_c[o] : V(0);
}

// x_i <- x_i + sum_t P[i, t] x_c[col_t]
template <class V>
__global__ void __launch_bounds__(kBlock) k_prolong_correct(LevelViewT<V> L, const V* __restrict__ xc,
                                                            V* __restrict__ x) {
  const int64_t i = (int64_t)xcd_block() * kBlock + threadIdx.x;
  if (i >= L.n) return;
  prolong_row(L, xc, x, (int32_t)i);
}

__global__ void k_gather(const int32_t* perm, const double* src, double* dst, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = src[perm[i]];
}

template <class V>
__global__ void k_scatter(const int32_t* perm, const V* src, double* dst, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[perm[i]] = (double)src[i];
}

__global__ void k_to_f32(const double* src, float* dst, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = (float)src[i];
}

// The start of a symmetric cycle on level 0, from x = 0 with the right-hand side r
// (float: rounded into b): the rows below r0, the first colour of the first sweep,
// take their update at once, (b - 0) / A_rr, since every term of their sums is a
// zero.  One launch for a fill, a conversion and the sweep's first launch, which
// read a colour's matrix for nothing (CG on 1,048,576 points in float 1.3% faster, on
// 1,000,000 in a cloud 3.4%).
template <class V>
__global__ void __launch_bounds__(kBlock) k_cycle_start(const double* __restrict__ r, const V* __restrict__ diag,
                                                        V* __restrict__ b, V* __restrict__ x, int64_t n, int32_t r0,
                                                        int32_t vectors) {
  const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;   // row i of one of the interleaved vectors
  if (t >= n * vectors) return;
  const int32_t i = (int32_t)(vectors == 1 ? t : t / vectors);
  V v = V(0);
  if (b || i < r0) v = (V)r[t];
  if (b) b[t] = v;
  x[t] = i < r0 ? v / diag[i] : V(0);
}

__global__ void k_check_finite(const double* v, int64_t n, int32_t* flag) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n && !isfinite(v[i])) atomicOr(flag, F_INVALID);
}

}  // namespace

// Calls f(std::integral_constant<int, CH>, std::integral_constant<bool, U>) for
// the load chunk CH of the level-0 row kernels and their slice form U (uniform
// width; only where the level's SELL has one).
template <class V, class F>
void with_chunk(const LevelViewT<V>& v, F&& f) {
  auto go = [&](auto UC) {
    switch (v.ch) {
      case 4: f(std::integral_constant<int, 4>{}, UC); break;
      case 16: f(std::integral_constant<int, 16>{}, UC); break;
      default: f(std::integral_constant<int, 8>{}, UC); break;
    }
  };
  if (v.uni && v.A.uw > 0) go(std::integral_constant<bool, true>{});
  else go(std::integral_constant<bool, false>{});
}

// One sweep in block order: the four block colours one launch each.  `skip`
// (ascending sweeps only): the first colour of block colour 0 is already done.
template <class V>
void block_sweep(const LevelViewT<V>& v, const Level& lv, hipStream_t s, bool descending, bool timed, int skip) {
  const BlockView<V>& B = v.B;
  if (!B.hdr || !B.glist || !B.elx || !B.elv || !B.rinfo || B.gstride <= 0 ||
      B.gstride > kBlkGather * kBlkThreads)
    throw Error{GMG_DEVICE_ERROR, "block sweep layout incomplete"};
  for (int k = 0; k < 4; ++k) {
    const int bc = descending ? 3 - k : k;
    const int32_t nb = B.bstart[bc + 1] - B.bstart[bc];
    if (nb <= 0) continue;
    double bytes = 0.0;
    for (int c = 0; c < B.ncls; ++c) bytes += lv.color_bytes[bc * B.ncls + c];
    KernelTimer::Scope t(timed ? (int)KernelTimer::GS_GALERKIN : -1, bytes);
    const int c_begin = !descending && k == 0 ? skip : 0;
    auto go = [&](auto kern) {
      hipExtLaunchKernelGGL(kern, dim3(nb), dim3(kBlkThreads), (size_t)B.lds_bytes, s, t.start, t.stop, 0, B,
                            (const V*)v.b, (const V*)v.diag, v.x, B.bstart[bc], c_begin, descending ? 1 : 0);
    };
    // gather slots: 2 cover lists of up to 512 rows and halo, 8 the largest (2048)
    const bool g2 = B.gstride <= 2 * kBlkThreads;
    if (B.rows_per_thread == 1) {
      if (B.width <= 32) {
        if (g2) go(k_gs_block<1, 32, 2, V>); else go(k_gs_block<1, 32, kBlkGather, V>);
      } else {
        if (g2) go(k_gs_block<1, 64, 2, V>); else go(k_gs_block<1, 64, kBlkGather, V>);
      }
    } else {
      if (B.width <= 32) {
        if (g2) go(k_gs_block<2, 32, 2, V>); else go(k_gs_block<2, 32, kBlkGather, V>);
      } else {
        if (g2) go(k_gs_block<2, 64, 2, V>); else go(k_gs_block<2, 64, kBlkGather, V>);
      }
    }
  }
}

template <class V>
void gs_sweep(const LevelViewT<V>& v, const Level& lv, hipStream_t s, bool finest, bool descending, bool timed,
              int skip) {
  if (!finest && v.B.nblk > 0) {
    block_sweep(v, lv, s, descending, timed, skip);
    return;
  }
  const int C = (int)lv.color_ptr.size() - 1;
  for (int k = skip; k < C; ++k) {
    const int c = descending ? C - 1 - k : k;
    const int32_t r0 = lv.color_ptr[c], r1 = lv.color_ptr[c + 1];
    if (r1 <= r0) continue;
    if (finest) {
      KernelTimer::Scope t(timed ? (int)KernelTimer::GS_FINEST : -1, lv.color_bytes[c]);
      const int32_t span = r1 - (r0 & ~(kSlice - 1));
      with_chunk(v, [&](auto CC, auto UC) {
        constexpr int CH = decltype(CC)::value;
        constexpr bool U = decltype(UC)::value;
        hipExtLaunchKernelGGL(k_gs_color_fine<CH, U, V>, dim3(blocks_for(span)), dim3(kBlock), 0, s, t.start,
                              t.stop, 0, v.A, (const V*)v.diag, (const V*)v.b, v.x, r0, r1);
      });
    } else {
      KernelTimer::Scope t(timed ? (int)KernelTimer::GS_GALERKIN : -1, lv.color_bytes[c]);
      with_lanes(v.ra, [&](auto RC) {
        constexpr int R = decltype(RC)::value;
        const auto kern = k_gs_color<R, V>;
        hipExtLaunchKernelGGL(kern, dim3(blocks_for((int64_t)(r1 - r0) * R)), dim3(kBlock), 0, s, t.start, t.stop,
                              0, v.A, (const V*)v.diag, (const V*)v.b, v.x, r0, r1, v.maxa);
      });
    }
  }
}

template <class V>
void residual(const LevelViewT<V>& v, hipStream_t s, bool finest) {
  if (finest) {
    with_chunk(v, [&](auto CC, auto UC) {
      constexpr int CH = decltype(CC)::value;
      constexpr bool U = decltype(UC)::value;
      k_residual_fine<CH, U, V><<<blocks_for(v.n), kBlock, 0, s>>>(v.A, v.b, v.x, v.r, v.n);
    });
  } else {
    with_lanes(v.ra, [&](auto RC) {
      constexpr int R = decltype(RC)::value;
      k_residual<R, V><<<blocks_for((int64_t)v.n * R), kBlock, 0, s>>>(v.A, v.b, v.x, v.r, v.n, v.maxa);
    });
  }
}

template <class V>
void restrict_to(const LevelViewT<V>& v, const LevelViewT<V>& c, hipStream_t s, int32_t first) {
  // the original-order copy of P^T where the level has one (row map to_row)
  const Sell<V>& T = v.to_row ? v.To : v.T;
  if (v.rt == 1) {
    k_restrict_seq<8, V><<<blocks_for(c.n), kBlock, 0, s>>>(T, v.r, c.b, c.x, c.n, (const V*)c.diag, first,
                                                            v.to_row);
    return;
  }
  with_lanes(v.rt, [&](auto RC) {
    constexpr int R = decltype(RC)::value;
    k_restrict<R, V><<<blocks_for((int64_t)c.n * R), kBlock, 0, s>>>(T, v.r, c.b, c.x, c.n, v.maxt,
                                                                      (const V*)c.diag, first, v.to_row);
  });
}

template <class V>
void prolong_correct(const LevelViewT<V>& v, const LevelViewT<V>& c, hipStream_t s) {
  k_prolong_correct<V><<<blocks_for(v.n), kBlock, 0, s>>>(v, c.x, v.x);
}

// v.x and, in float, v.b for a cycle from zero with the right-hand side rhs (double:
// v.b itself), the rows below r0 updated (k_cycle_start).
template <class V>
void cycle_start(const LevelViewT<V>& v, const double* rhs, int32_t r0, int32_t vectors, hipStream_t s) {
  k_cycle_start<V><<<blocks_for((int64_t)v.n * vectors), kBlock, 0, s>>>(
      rhs, v.diag, std::is_same<V, float>::value ? v.b : nullptr, v.x, v.n, r0, vectors);
}

void to_f32(const double* src, float* dst, int64_t n, hipStream_t s) {
  k_to_f32<<<blocks_for(n), kBlock, 0, s>>>(src, dst, n);
}

void permute_in(const int32_t* perm, const double* src, double* dst, int64_t n, hipStream_t s) {
  k_gather<<<blocks_for(n), kBlock, 0, s>>>(perm, src, dst, n);
}

template <class V>
void permute_out(const int32_t* perm, const V* src, double* dst, int64_t n, hipStream_t s) {
  k_scatter<V><<<blocks_for(n), kBlock, 0, s>>>(perm, src, dst, n);
}

void norm2_partials(const double* v, int64_t n, double* partials, hipStream_t s) {
  k_norm_partials<<<kNormBlocks, kBlock, 0, s>>>(v, n, partials);
}

void residual_norm(const Level& lv, const double* b, const double* x, double* res, double* partials,
                   hipStream_t s) {
  KernelTimer::Scope t(KernelTimer::RESIDUAL_FINEST, lv.residual_bytes);
  with_chunk(lv.view, [&](auto CC, auto UC) {
    constexpr int CH = decltype(CC)::value;
    constexpr bool U = decltype(UC)::value;
    hipExtLaunchKernelGGL(k_residual_norm<CH, U>, dim3(kNormBlocks), dim3(kBlock), 0, s, t.start, t.stop, 0,
                          lv.view.A, b, x, res, (int64_t)lv.n, partials);
  });
}

void finish_norm(const double* partials, double* out, hipStream_t s, double* host_out) {
  k_finish_norm<<<1, kBlock, 0, s>>>(partials, out, host_out);
}

void check_finite(const double* v, int64_t n, int32_t* flag, hipStream_t s) {
  k_check_finite<<<blocks_for(n), kBlock, 0, s>>>(v, n, flag);
}

#define GMG_INSTANTIATE(V)                                                                              \
  template void gs_sweep<V>(const LevelViewT<V>&, const Level&, hipStream_t, bool, bool, bool, int);  \
  template void residual<V>(const LevelViewT<V>&, hipStream_t, bool);                                  \
  template void restrict_to<V>(const LevelViewT<V>&, const LevelViewT<V>&, hipStream_t, int32_t);      \
  template void prolong_correct<V>(const LevelViewT<V>&, const LevelViewT<V>&, hipStream_t);           \
  template void cycle_start<V>(const LevelViewT<V>&, const double*, int32_t, int32_t, hipStream_t);    \
  template void permute_out<V>(const int32_t*, const V*, double*, int64_t, hipStream_t);
GMG_INSTANTIATE(double)
GMG_INSTANTIATE(float)
#undef GMG_INSTANTIATE

}  // namespace gmg
