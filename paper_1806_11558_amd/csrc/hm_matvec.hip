// H-matrix-vector products y = H x and y = H^T x (Sec. 2.3, last paragraph:
// dense leaves apply their stored block, admissible leaves the low-rank
// factors), with every output row owned by exactly one workgroup: no atomics,
// a fixed summation order, bitwise reproducible results.
//
// Storage (built by the setup):
//   row panels  for every row leaf c, its dense slices and (per ACA chunk) its
//               U slices are each one contiguous column-major panel
//               ld_c x W; column j of a panel multiplies z[colmap[col0 + j]]
//               where z = [x in Morton order ; t]
//   V blocks    the V factor of every admissible block is contiguous: its
//               column-leaf slices (ld x r, column-major) one after another
//
//   forward     z[0..n)      = x[perm]                          (gather)
//               z[n + toff_b + l] = sum_i V_b[i][l] x_sigma[i] (one wavefront
//                                                               per block)
//               y_c = sum over the row panels of c of  P z[map]  (per leaf)
//   transposed  w[col] = sum_i P[i][col] x_c[i] for every panel column
//               (per row leaf), s_b[l] = sum over the row leaves of b of the
//               w of its U columns (per block), then per column leaf
//               y_c = sum over dense blocks of the w entries of its columns
//                   + sum over its V slices of V s_b
//
// A wavefront reads a slice in 16-byte granules: lane = (column group cg,
// row granule g), R = ld/G row granules per column, C = 64/R columns per
// instruction.
#include <type_traits>

#include "hm_internal.h"
#include "hm_wave.h"

namespace hm {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));

// Granule loads of G stored values per lane, returned in the arithmetic type
// E; the stored operator is streamed once per product, so the loads are
// non-temporal.  FP32 and FP16 granules both cover 4 rows (16 and 8 bytes),
// so dense and FP16 factor panels of a leaf share one lane layout.
template <typename T>
struct Gran;
template <>
struct Gran<float> {
  using E = float;
  static constexpr int G = 4;
  __device__ static inline void load(const float* p, float* o) {
    const f32x4 v = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p));
    o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w;
  }
};
template <>
struct Gran<double> {
  using E = double;
  static constexpr int G = 2;
  __device__ static inline void load(const double* p, double* o) {
    const f64x2 v = __builtin_nontemporal_load(reinterpret_cast<const f64x2*>(p));
    o[0] = v.x; o[1] = v.y;
  }
};
template <>
struct Gran<_Float16> {
  using E = float;
  static constexpr int G = 4;
  __device__ static inline void load(const _Float16* p, float* o) {
    const f16x4 v = __builtin_nontemporal_load(reinterpret_cast<const f16x4*>(p));
    o[0] = (float)v.x; o[1] = (float)v.y; o[2] = (float)v.z; o[3] = (float)v.w;
  }
};

// NR consecutive values z[0..NR) (16-byte aligned when NR * sizeof(A) is a
// multiple of 16: z rows are NR values long and the buffer is 256-byte aligned).
template <typename A, int NR>
__device__ inline void load_row(const A* __restrict__ p, A (&o)[NR]) {
  if constexpr (sizeof(A) == 8 && NR % 2 == 0) {
#pragma unroll
    for (int k = 0; k < NR; k += 2) {
      const f64x2 v = *reinterpret_cast<const f64x2*>(p + k);
      o[k] = v.x;
      o[k + 1] = v.y;
    }
  } else if constexpr (sizeof(A) == 4 && NR % 4 == 0) {
#pragma unroll
    for (int k = 0; k < NR; k += 4) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(p + k);
      o[k] = v.x;
      o[k + 1] = v.y;
      o[k + 2] = v.z;
      o[k + 3] = v.w;
    }
  } else {
#pragma unroll
    for (int k = 0; k < NR; ++k) o[k] = p[k];
  }
}

// Sum of v over the R lanes g = 0..R-1 of a lane segment; valid in the lane
// with g == 0.  Every lane of the wavefront must call it.
template <typename A>
__device__ inline A seg_sum(A v, int g, int R) {
  for (int s = 1; s < R; s <<= 1) {
    const A o = __shfl_down(v, s, 64);
    if (g + s < R) v += o;
  }
  return v;
}

// Workgroup w runs on XCD w mod 8 (8 XCDs, each with its own L2).  Logical
// index li -> item (li mod 8) * per + li / 8 gives every XCD a contiguous
// range of leaves, so neighbouring leaves, which
// gather mostly the same x and t values, share one L2.  A bijection of
// [0, 8 per) onto itself; items >= the count are skipped.
__device__ inline int64_t xcd_item(int64_t li, int64_t per) {
  return (li % kXcds) * per + li / kXcds;
}

// ------------------------------------------------------------------ gather
template <typename VT, typename A>
__global__ void k_gather(const VT* __restrict__ x, int nrhs, int k0, int nr,
                         const int32_t* __restrict__ perm, int64_t n, A* __restrict__ z) {
  const int64_t tot = n * nr;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < tot;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t p = e / nr;
    const int k = (int)(e % nr);
    z[e] = (A)x[(int64_t)perm[p] * nrhs + k0 + k];
  }
}

// ------------------------------------------------------------------ forward, phase 1
// One wavefront per admissible block: t_b = V_b^T x_sigma (times the U scale
// when the factors are FP16), written to z[n + toff + l].
//
// Lane = (column group cg, row granule g); the P = ceil(r / C) passes of C
// columns each keep a register accumulator.  When all column-leaf slices
// share one ld (the usual case) the x granule is loaded once per slice, the
// accumulators run over all slices, and each pass is reduced once at the
// end; otherwise every slice is reduced on its own.  Column sums move to
// lane l, which owns term l.
template <typename A, int NR>
__device__ inline void fwd1_flush(A (&p)[NR], int g, int R, int j0, int C, int r, int lane,
                                  A (&tl)[NR]) {
#pragma unroll
  for (int k = 0; k < NR; ++k) p[k] = seg_sum(p[k], g, R);
  const int q = lane - j0;
  const bool mine = q >= 0 && q < C && lane < r;
  const int src = mine ? q * R : 0;
#pragma unroll
  for (int k = 0; k < NR; ++k) {
    const A v = __shfl(p[k], src, 64);
    if (mine) tl[k] += v;
  }
}

// The slices of one block with every column-leaf slice of ld rows: P passes
// of C columns, P known at compile time so that the granules of all passes
// are loaded with no branch between them and the x loads; columns past r
// read column r - 1 into accumulators that are never flushed.
template <typename T, typename A, int NR, int P>
__device__ inline void fwd1_uniform(const VUnit& M, const MvLeaves& L, const A* __restrict__ z,
                                    int r, int ld, int R, int C, int cg, int g, bool act, int lane,
                                    A (&tl)[NR]) {
  constexpr int G = Gran<T>::G;
  A acc[P][NR];
#pragma unroll
  for (int q = 0; q < P; ++q)
#pragma unroll
    for (int k = 0; k < NR; ++k) acc[q][k] = 0;
  // 32-bit element offsets of the lane's granule in each pass
  int off[P];
#pragma unroll
  for (int q = 0; q < P; ++q) off[q] = min(q * C + cg, r - 1) * ld + g * G;
  const int sstride = ld * M.vw;
  const T* Sl = reinterpret_cast<const T*>((uintptr_t)M.vptr);
  int lo = L.lo[M.sf];                       // the leaves of sigma are consecutive
  for (int lf = M.sf; lf <= M.sl; ++lf, Sl += sstride) {
    const int m = L.m[lf];
    typename Gran<T>::E sv[P][G];
#pragma unroll
    for (int q = 0; q < P; ++q) Gran<T>::load(Sl + off[q], sv[q]);
    A xg[G][NR];
#pragma unroll
    for (int e = 0; e < G; ++e) {
      // unconditional load of a clamped row, zeroed outside the slice
      const int row = g * G + e;
      const bool in = act && row < m;
      const A* zr = z + (int64_t)(lo + (in ? row : 0)) * NR;
#pragma unroll
      for (int k = 0; k < NR; ++k) {
        const A v = zr[k];
        xg[e][k] = in ? v : (A)0;
      }
    }
#pragma unroll
    for (int q = 0; q < P; ++q)
#pragma unroll
      for (int e = 0; e < G; ++e)
#pragma unroll
        for (int k = 0; k < NR; ++k) acc[q][k] += (A)sv[q][e] * xg[e][k];
    lo += m;
  }
#pragma unroll
  for (int q = 0; q < P; ++q) fwd1_flush<A, NR>(acc[q], g, R, q * C, C, r, lane, tl);
}

// Wavefronts per SIMD: all eight (64 registers), but for the 16 accumulators
// of two columns of FP16 slices, which take up to 128.
template <typename T, typename A, int NR>
constexpr int fwd1_waves() {
  return NR == 2 && sizeof(T) == 2 ? 4 : 8;
}

template <typename T, typename A, int NR>
__global__ __launch_bounds__(256, (fwd1_waves<T, A, NR>())) void k_fwd1(
    const VUnit* __restrict__ meta, int64_t nl, MvLeaves L, A* __restrict__ z, int64_t n,
    const float* __restrict__ su) {
  constexpr int G = Gran<T>::G;
  static_assert(NR <= 2, "more right-hand sides go to the matrix cores");
  // loads per lane of the one-pass form: the phase-1 units of FP16 slices are
  // sized for eight, of FP32 and FP64 ones for four; a unit with more passes
  // than this would reduce every slice on its own (FP16, 2 columns, N =
  // 81,920, leaf 64: phase 1 394 us with four, 82 with eight)
  constexpr int PMAX = sizeof(T) == 2 ? 8 : 4;
  const int lane = threadIdx.x & 63;
  // wave-uniform block index: descriptors and leaf data come in by scalar loads
  const int64_t wid = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t nw = (int64_t)gridDim.x * 4;
  // the next block's descriptor is loaded one iteration ahead
  VUnit Mn;
  if (wid < nl) Mn = meta[wid];
  for (int64_t b = wid; b < nl; b += nw) {
    const VUnit M = Mn;
    if (b + nw < nl) Mn = meta[b + nw];
    const int r = M.r;
    if (r == 0) continue;
    A tl[NR];
#pragma unroll
    for (int k = 0; k < NR; ++k) tl[k] = 0;
    const T* S = reinterpret_cast<const T*>((uintptr_t)M.vptr);
    const int R0 = M.vld / G, C0 = R0 > 0 ? 64 / R0 : 1;
    if (M.vld > 0 && r <= PMAX * C0 && r <= 64) {
      const int ld = M.vld, R = R0, C = C0;
      // lane / R by a multiply and shift (exact for lane < 64, R <= 64)
      const unsigned mul = (unsigned)(65536.0f / (float)R) + 1u;
      const int cg = (int)(((unsigned)lane * mul) >> 16), g = lane - cg * R;
      const bool act = cg < C;
      const int P = (r + C - 1) / C;
      switch (P) {                                      // uniform over the wavefront
        case 1: fwd1_uniform<T, A, NR, 1>(M, L, z, r, ld, R, C, cg, g, act, lane, tl); break;
        case 2: fwd1_uniform<T, A, NR, 2>(M, L, z, r, ld, R, C, cg, g, act, lane, tl); break;
        case 3: fwd1_uniform<T, A, NR, 3>(M, L, z, r, ld, R, C, cg, g, act, lane, tl); break;
        case 4: fwd1_uniform<T, A, NR, 4>(M, L, z, r, ld, R, C, cg, g, act, lane, tl); break;
        case 5:
          if constexpr (PMAX >= 5) fwd1_uniform<T, A, NR, 5>(M, L, z, r, ld, R, C, cg, g, act, lane, tl);
          break;
        case 6:
          if constexpr (PMAX >= 6) fwd1_uniform<T, A, NR, 6>(M, L, z, r, ld, R, C, cg, g, act, lane, tl);
          break;
        case 7:
          if constexpr (PMAX >= 7) fwd1_uniform<T, A, NR, 7>(M, L, z, r, ld, R, C, cg, g, act, lane, tl);
          break;
        default:
          if constexpr (PMAX >= 8) fwd1_uniform<T, A, NR, 8>(M, L, z, r, ld, R, C, cg, g, act, lane, tl);
          break;
      }
    } else {
      // general path, 64 terms (one per lane) at a time
      for (int t0 = 0; t0 < r; t0 += 64) {
        const int rc = min(64, r - t0);
        const T* Sl = S;
#pragma unroll
        for (int k = 0; k < NR; ++k) tl[k] = 0;
        for (int lf = M.sf; lf <= M.sl; ++lf) {
          const int ld = (int)(L.ldpre[lf + 1] - L.ldpre[lf]);
          const int R = ld / G, C = 64 / R;
          const int cg = lane / R, g = lane % R;
          const bool act = cg < C;
          const int m = L.m[lf], lo = L.lo[lf];
          A xg[G][NR];
#pragma unroll
          for (int e = 0; e < G; ++e) {
            const int row = g * G + e;
#pragma unroll
            for (int k = 0; k < NR; ++k)
              xg[e][k] = (act && row < m) ? z[(int64_t)(lo + row) * NR + k] : (A)0;
          }
          for (int j0 = 0; j0 < rc; j0 += C) {
            const int j = j0 + cg;
            A p[NR];
#pragma unroll
            for (int k = 0; k < NR; ++k) p[k] = 0;
            if (act && j < rc) {
              typename Gran<T>::E sv[G];
              Gran<T>::load(Sl + (int64_t)(t0 + j) * ld + g * G, sv);
#pragma unroll
              for (int e = 0; e < G; ++e)
#pragma unroll
                for (int k = 0; k < NR; ++k) p[k] += (A)sv[e] * xg[e][k];
            }
            fwd1_flush<A, NR>(p, g, R, j0, C, rc, lane, tl);
          }
          Sl += (int64_t)ld * M.vw;
        }
        if (t0 + 64 < r && lane < rc) {       // every chunk but the last one
          const A sc = su ? (A)su[M.toff + t0 + lane] : (A)1;
#pragma unroll
          for (int k = 0; k < NR; ++k) z[(n + M.toff + t0 + lane) * NR + k] = tl[k] * sc;
        }
      }
    }
    // terms 64 q + lane of the last chunk q (the only chunk when r <= 64)
    const int tlast = r > 64 ? (r - 1) / 64 * 64 : 0;
    if (tlast + lane < r) {
      const A sc = su ? (A)su[M.toff + tlast + lane] : (A)1;
#pragma unroll
      for (int k = 0; k < NR; ++k) z[(n + M.toff + tlast + lane) * NR + k] = tl[k] * sc;
    }
  }
}

// ------------------------------------------------------------------ forward, phase 2
// Per row leaf: y_c = sum over its panels of P z[colmap], then scattered to
// application order.  Panel 0 of a leaf holds dense slices (type TD), the
// others U slices (type TL); both share the lane layout.
//
// The workgroup first gathers the z values of a tile of panel columns into
// LDS (one load per column instead of one per lane, and no map -> z
// dependency inside the streaming loop), then streams the tile's columns:
// wavefront w takes column groups w, w + 4, ..., UNR of them at a time.
// Loads are unconditional: a lane without a column of its own reads the
// panel's last column and contributes zero, so the compiler keeps all UNR
// loads in flight instead of waiting inside divergent branches.  A tile
// holds kZTileBytes of z.
constexpr int kZTileBytes = 8192;
template <typename A, int NR>
constexpr int z_tile() { return kZTileBytes / (int)(NR * sizeof(A)); }

template <typename T, typename A, int NR, int G>
__device__ inline void fwd2_run_lds(const Unit& U, int ld, int C, int cg, int g,
                                    bool act, int wave, const int32_t* __restrict__ colmap,
                                    const A* __restrict__ z, A* __restrict__ zt,
                                    A (&acc)[G][NR]) {
  constexpr int UNR = 4;
  static_assert(Gran<T>::G == G, "panel granules must cover the same rows");
  const int uw = U.w;
  const T* S = reinterpret_cast<const T*>((uintptr_t)U.data) + g * G;
  const int32_t* map = colmap + U.col;
  constexpr int kTile = z_tile<A, NR>();
  for (int t0 = 0; t0 < uw; t0 += kTile) {
    const int tw = min(kTile, uw - t0);
    __syncthreads();                                   // the previous tile is consumed
    for (int c = threadIdx.x; c < tw; c += blockDim.x) {
      A v[NR];
      load_row<A, NR>(z + (int64_t)map[t0 + c] * NR, v);
#pragma unroll
      for (int k = 0; k < NR; ++k) zt[c * NR + k] = v[k];
    }
    __syncthreads();
    const T* St = S + (int64_t)t0 * ld;
    const int ngrp = (tw + C - 1) / C;
    for (int q0 = wave; q0 < ngrp; q0 += 4 * UNR) {
      typename Gran<T>::E s[UNR][G];
      int jl[UNR];
      bool ok[UNR];
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        const int q = q0 + 4 * u;
        const int j = q * C + cg;
        ok[u] = act && q < ngrp && j < tw;
        jl[u] = ok[u] ? j : tw - 1;
        Gran<T>::load(St + (int64_t)jl[u] * ld, s[u]);
      }
      // all loads before the first wait, only LDS reads may pass them: 148 leaves of
      // 39 rows, FP32, two double columns 51.3 -> 48.2 us; N = 81,920, leaf 64,
      // 624 -> 605, four columns 638 -> 610
      __builtin_amdgcn_sched_barrier(0x100);
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
#pragma unroll
        for (int e = 0; e < G; ++e) {
          const A sv = ok[u] ? (A)s[u][e] : (A)0;
#pragma unroll
          for (int k = 0; k < NR; ++k) acc[e][k] += sv * zt[jl[u] * NR + k];
        }
      }
    }
  }
}

// Two columns of factors narrower than the vectors: conversions in flight take
// registers, and without a bound there are four wavefronts per SIMD instead of
// six; N = 40,500, leaf 16, FP32, double vectors 481 -> 459 us, 5,780, leaf 64,
// 49.9 -> 46.9.  (One column with all eight: 334 -> 327 us, but 3,380 elements,
// 64 leaves, 30.2 -> 31.8 and FP16 30.6 -> 32.5.)
template <typename TL, typename A, int NR>
constexpr int fwd2_waves() { return sizeof(TL) < sizeof(A) && NR == 2 ? 6 : 1; }
template <typename TD, typename TL, typename A, int NR>
__global__ __launch_bounds__(256, (fwd2_waves<TL, A, NR>())) void k_fwd2(
    const Unit* __restrict__ units, int64_t nunits, const int32_t* __restrict__ colmap,
    const A* __restrict__ z, A* __restrict__ ypart, int ldmax) {
  constexpr int G = Gran<TD>::G;
  __shared__ A ybuf[4][kMaxLeaf][NR];
  __shared__ A zt[z_tile<A, NR>() * NR];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t per = (nunits + kXcds - 1) / kXcds;
  for (int64_t li = blockIdx.x; li < per * kXcds; li += gridDim.x) {
    const int64_t u = xcd_item(li, per);
    if (u >= nunits) continue;                          // uniform over the workgroup
    const Unit U = units[u];
    const int ld = U.ld, m = U.m;
    const int R = ld / G, C = 64 / R;
    const int cg = lane / R, g = lane % R;
    const bool act = cg < C;
    A acc[G][NR];
#pragma unroll
    for (int e = 0; e < G; ++e)
#pragma unroll
      for (int k = 0; k < NR; ++k) acc[e][k] = 0;
    if (std::is_same<TD, TL>::value || U.dense)
      fwd2_run_lds<TD, A, NR, G>(U, ld, C, cg, g, act, wave, colmap, z, zt, acc);
    else
      fwd2_run_lds<TL, A, NR, G>(U, ld, C, cg, g, act, wave, colmap, z, zt, acc);
    // combine the column groups (tree over cg, stride R), then the waves
#pragma unroll
    for (int e = 0; e < G; ++e)
#pragma unroll
      for (int k = 0; k < NR; ++k) {
        A v = acc[e][k];
        for (int s = 1; s < C; s <<= 1) {
          const A o = __shfl_down(v, s * R, 64);
          if (cg + s < C) v += o;
        }
        acc[e][k] = v;
      }
    if (cg == 0) {
#pragma unroll
      for (int e = 0; e < G; ++e) {
        const int row = g * G + e;
        if (row < kMaxLeaf)
#pragma unroll
          for (int k = 0; k < NR; ++k) ybuf[wave][row][k] = acc[e][k];
      }
    }
    __syncthreads();
    A* yp = ypart + u * ldmax * NR;
    for (int e = threadIdx.x; e < m * NR; e += blockDim.x) {
      const int row = e / NR, k = e % NR;
      yp[e] = ((ybuf[0][row][k] + ybuf[1][row][k]) + ybuf[2][row][k]) + ybuf[3][row][k];
    }
    __syncthreads();
  }
}

// y rows of every leaf = sum of its units' partial rows (in unit order),
// scattered to application order.  One wavefront per leaf for one or two
// right-hand sides (a leaf has at most 64 rows), a workgroup for more: a
// leaf of 40 rows has 640 sums of 16 columns, ten dependent rounds for one
// wavefront (2,048 leaves of FP64 sums, 16 columns: 93 -> 35 us).
template <int NR>
constexpr int sum_leaves() { return NR <= 2 ? 4 : 1; }   // leaves per 256-thread workgroup
template <typename A, typename VT, int NR>
__global__ __launch_bounds__(256) void k_fwd2_sum(MvLeaves L, const int32_t* __restrict__ ubeg,
                                                  const A* __restrict__ ypart, int ldmax,
                                                  const int32_t* __restrict__ perm,
                                                  VT* __restrict__ y, int nrhs, int k0, int nv) {
  constexpr int LW = sum_leaves<NR>(), TL = 256 / LW;
  for (int64_t c = blockIdx.x * LW + threadIdx.x / TL; c < L.nleaf; c += (int64_t)gridDim.x * LW) {
    const int m = L.m[c], lo = L.lo[c];
    const int u0 = ubeg[c], u1 = ubeg[c + 1];
    for (int e = threadIdx.x % TL; e < m * NR; e += TL) {
      const int row = e / NR, k = e % NR;
      A v = 0;
      for (int u = u0; u < u1; ++u) v += ypart[(int64_t)u * ldmax * NR + e];
      if (k < nv) y[(int64_t)perm[lo + row] * nrhs + k0 + k] = (VT)v;
    }
  }
}

// ------------------------------------------------------------------ many right-hand sides on MFMA
// With many right-hand sides, both forward phases are small dense
// products with a long inner dimension (phase 1 from 4 columns on, phase 2
// from 8): phase 1 is T_b = V_b^T X (terms x
// right-hand sides, inner dimension = rows of sigma), phase 2 is
// Y_c += P Z (rows of the leaf x right-hand sides, inner dimension = panel
// columns).  Both run on 16 x 16 x 4 matrix instructions, C[16][16] +=
// A[16][4] B[4][16] with, for lane l, a = A[l % 16][l / 16] and
// b = B[l / 16][l % 16]: v_mfma_f64_16x16x4 for double vectors (item j of
// the accumulator = C[4 j + l / 16][l % 16]), v_mfma_f32_16x16x4 for float
// vectors (item j = C[4 (l / 16) + j][l % 16]).  Stored values are widened
// to the accumulation type, double or float as on the vector path.
typedef double f64x4 __attribute__((ext_vector_type(4)));

__device__ inline f64x4 mfma16(double a, double b, f64x4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ inline f32x4 mfma16(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
template <typename A>
struct Mfma;
template <>
struct Mfma<double> {
  using V = f64x4;
  // row of accumulator item j in lane group q = l / 16
  __device__ static inline int row(int j, int q) { return 4 * j + q; }
};
template <>
struct Mfma<float> {
  using V = f32x4;
  __device__ static inline int row(int j, int q) { return 4 * q + j; }
};

// N consecutive stored values (4, 2 or 1; the address is a multiple of their
// size, 16 bytes for four doubles).  Panel addresses come from descriptors,
// so the compiler would read them by flat instructions, which count as LDS
// accesses too: every wait for an LDS result would then wait for all panel
// loads in flight.  The cast to the global address space keeps the two apart.
// NT: non-temporal.
template <typename T, int N, bool NT>
__device__ inline void load_n(const T* p, T* o) {
  if constexpr (N * sizeof(T) > 16) {
    load_n<T, N / 2, NT>(p, o);
    load_n<T, N / 2, NT>(p + N / 2, o + N / 2);
  } else if constexpr (N == 1) {
    const __attribute__((address_space(1))) T* q = (const __attribute__((address_space(1))) T*)p;
    o[0] = NT ? __builtin_nontemporal_load(q) : *q;
  } else {
    typedef T TV __attribute__((ext_vector_type(N)));
    const __attribute__((address_space(1))) TV* q = (const __attribute__((address_space(1))) TV*)p;
    const TV u = NT ? __builtin_nontemporal_load(q) : *q;
#pragma unroll
    for (int e = 0; e < N; ++e) o[e] = u[e];
  }
}
// The element i past a wavefront-uniform base, i of 32 bits: base in scalar
// registers, one vector offset.
template <typename T>
__device__ inline const T* at32(const T* base, uint32_t i) {
  return reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) +
                                    (size_t)(i * (uint32_t)sizeof(T)));
}

// ------------------------------------------------------------------ gather, 4 to 16 right-hand sides
// One workgroup per leaf writes its x twice: row by row into z (the form the
// panel columns of phase 2 pick single rows from) and, transposed, into xt:
// leaf c holds NR columns of ld_c values at xt + ldpre[c] NR, rows in [m, ld)
// zero, so that phase 1 reads four rows of one right-hand side with one load
// and needs no row masks.  Columns nv .. NR - 1 (a pass wider than what is
// left) are zero.  z may be null.
template <typename VT, typename A, int NR>
__global__ __launch_bounds__(256) void k_gather_x(const VT* __restrict__ x, int nrhs, int k0,
                                                  int nv, const int32_t* __restrict__ perm,
                                                  MvLeaves L, A* __restrict__ z,
                                                  A* __restrict__ xt) {
  for (int64_t c = blockIdx.x; c < L.nleaf; c += gridDim.x) {
    const int m = L.m[c], lo = L.lo[c];
    const int ld = (int)(L.ldpre[c + 1] - L.ldpre[c]);
    A* xc = xt + L.ldpre[c] * NR;
    for (int e = threadIdx.x; e < ld * NR; e += blockDim.x) {
      const int i = e / NR, k = e % NR;
      const A v = (i < m && k < nv) ? (A)x[(int64_t)perm[lo + min(i, m - 1)] * nrhs + k0 + min(k, nv - 1)] : (A)0;
      if (z && i < m) z[(int64_t)(lo + i) * NR + k] = v;
      xc[k * ld + i] = v;
    }
  }
}

// ------------------------------------------------------------------ phase 1 on MFMA
// One wavefront per unit of up to 64 terms (four tiles of 16).  The inner
// dimension (rows) may be summed in any order: lane (term lr, quad lq) reads
// the ST consecutive rows i0 + ST lq .. of its term with one load and feeds
// them to ST instructions, and the x values of its right-hand side come from
// the transposed copy in the same form.  The rows of a leaf are its ld:
// tiles of 16 (ST = 4), then one of 8 (ST = 2) and one of 4 (ST = 1) for the
// rest of ld (a multiple of 4), so nothing is spent on padding beyond ld, and
// no load or product has a mask: rows in [m, ld) are zero on both sides, and
// terms past r - 1 repeat term r - 1 into rows of the result that are not
// stored.  The loads are temporal: a term's rows are 16 to 128 bytes per tile,
// pieces of a cache line whose rest the next tile needs (non-temporal, FP64
// fetched 3.3 GB for 1.8 GB of factors).  16 columns at N = 81,920, FP64 581 ->
// 440 us, FP32 281 -> 229; FP16 at N = 162,000 551 -> 272 us; four columns, FP32,
// 1,458 -> 212 us (on the vector units before).  Bound by HBM in FP64: by the
// counters 2.7 GB (z and lines read again with the 1.8 of factors) at 6.3 TB/s;
// FP32 5.5, FP16 4.5 TB/s, the matrix cores busy for a fifth to a third.
template <typename T, typename A, int NTL, int ST, int IU>
__device__ inline void fwd1x_rows(const T* __restrict__ S, const A* __restrict__ xb, int ld,
                                  int i0, const int (&tc)[NTL], int xo, int lq,
                                  typename Mfma<A>::V (&acc)[4]) {
  T av[IU][NTL][ST];
  A bv[IU][ST];
#pragma unroll
  for (int u = 0; u < IU; ++u) {
    const int i = i0 + 16 * u + ST * lq;
#pragma unroll
    for (int t = 0; t < NTL; ++t) load_n<T, ST, false>(S + (tc[t] * ld + i), av[u][t]);
    load_n<A, ST, false>(xb + (xo * ld + i), bv[u]);
  }
#pragma unroll
  for (int u = 0; u < IU; ++u)
#pragma unroll
    for (int e = 0; e < ST; ++e)
#pragma unroll
      for (int t = 0; t < NTL; ++t) acc[t] = mfma16((A)av[u][t][e], bv[u][e], acc[t]);
}

// All rows of one leaf: the columns tc of the slice S against the leaf's x.
template <typename T, typename A, int NTL>
__device__ inline void fwd1x_leaf(const T* __restrict__ S, const A* __restrict__ xb, int ld,
                                  const int (&tc)[NTL], int xo, int lq,
                                  typename Mfma<A>::V (&acc)[4]) {
  // tiles of 16 rows, two at a time where their registers fit
  constexpr int IU = sizeof(T) == 8 ? 1 : 2;
  int i0 = 0;
  for (; i0 + 16 * IU <= ld; i0 += 16 * IU)
    fwd1x_rows<T, A, NTL, 4, IU>(S, xb, ld, i0, tc, xo, lq, acc);
  if (IU == 2 && i0 + 16 <= ld) {
    fwd1x_rows<T, A, NTL, 4, 1>(S, xb, ld, i0, tc, xo, lq, acc);
    i0 += 16;
  }
  if (ld & 8) {
    fwd1x_rows<T, A, NTL, 2, 1>(S, xb, ld, i0, tc, xo, lq, acc);
    i0 += 8;
  }
  if (ld & 4) fwd1x_rows<T, A, NTL, 1, 1>(S, xb, ld, i0, tc, xo, lq, acc);
}

template <typename T, typename A, int NR, int NTL>
__device__ inline void fwd1x_pass(const VUnit& M, const MvLeaves& L, const A* __restrict__ xt,
                                  int tg, int r, int lr, int lq,
                                  typename Mfma<A>::V (&acc)[4]) {
  const T* S = reinterpret_cast<const T*>((uintptr_t)M.vptr);
  int tc[NTL];                            // clamped term of each tile
#pragma unroll
  for (int t = 0; t < NTL; ++t) tc[t] = min(tg + t * 16 + lr, r - 1);
  const int xo = lr & (NR - 1);           // NR < 16: columns repeat, not stored
  int64_t lp = L.ldpre[M.sf];
  for (int lf = M.sf; lf <= M.sl; ++lf) {
    const int64_t lpn = L.ldpre[lf + 1];
    const int ld = (int)(lpn - lp);
    fwd1x_leaf<T, A, NTL>(S, xt + lp * NR, ld, tc, xo, lq, acc);
    S += (int64_t)ld * M.vw;
    lp = lpn;
  }
}

// Calls put(row, rhs, value) for the rows and right-hand sides of a 16-row
// result tile.  In double and for 16 columns the lanes of one call already
// lie side by side in memory; with fewer float columns a call per item would
// write 16- or 32-byte pieces, so the items are exchanged first and a call
// covers 16 / NR of the four rows of every quad.
template <typename A, int NR, typename Put>
__device__ inline void tile_out(const typename Mfma<A>::V& acc, int lr, int lq, const Put& put) {
  if constexpr (sizeof(A) == 8 || NR == 16) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (lr < NR) put(Mfma<A>::row(j, lq), lr, acc[j]);
  } else {
    constexpr int GR = NR < 4 ? 4 : 16 / NR;     // rows per call
    const int g = lr / NR, k = lr & (NR - 1);
#pragma unroll
    for (int h = 0; h < 4; h += GR) {
      A v = 0;
#pragma unroll
      for (int q = 0; q < GR; ++q) {
        const A o = __shfl(acc[h + q], lq * 16 + k, 64);
        v = g == q ? o : v;
      }
      if (g < GR) put(4 * lq + h + g, k, v);
    }
  }
}

template <typename T, typename A, int NR>
__global__ __launch_bounds__(256) void k_fwd1x(const VUnit* __restrict__ meta, int64_t nl,
                                               MvLeaves L, const A* __restrict__ xt,
                                               A* __restrict__ zt, int64_t n,
                                               const float* __restrict__ su) {
  using V = typename Mfma<A>::V;
  static_assert(NR == 4 || NR == 8 || NR == 16, "MFMA phase 1 takes 4, 8 or 16 right-hand sides");
  const int lane = threadIdx.x & 63;
  const int lr = lane & 15, lq = lane >> 4;     // a: term lr, row lq; b: row lq, rhs lr
  const int64_t wid = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t nw = (int64_t)gridDim.x * 4;
  for (int64_t b = wid; b < nl; b += nw) {
    const VUnit M = meta[b];
    const int r = M.r;
    if (r == 0) continue;
    for (int tg = 0; tg < r; tg += 64) {
      const int ntile = min(4, (r - tg + 15) / 16);
      V acc[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) acc[t] = V{0, 0, 0, 0};
      switch (ntile) {                        // uniform over the wavefront
        case 1: fwd1x_pass<T, A, NR, 1>(M, L, xt, tg, r, lr, lq, acc); break;
        case 2: fwd1x_pass<T, A, NR, 2>(M, L, xt, tg, r, lr, lq, acc); break;
        case 3: fwd1x_pass<T, A, NR, 3>(M, L, xt, tg, r, lr, lq, acc); break;
        default: fwd1x_pass<T, A, NR, 4>(M, L, xt, tg, r, lr, lq, acc); break;
      }
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        if (t < ntile) {
          tile_out<A, NR>(acc[t], lr, lq, [&](int row, int k, A v) {
            const int term = tg + t * 16 + row;
            if (term < r) {
              const A sc = su ? (A)su[M.toff + term] : (A)1;
              zt[(n + M.toff + term) * NR + k] = v * sc;
            }
          });
        }
      }
    }
  }
}

// ------------------------------------------------------------------ phase 2 on MFMA
// A leaf of ld rows takes NT = ceil(ld / 16) row tiles.  Lane (i = lr, column
// lq of a quad) reads its rows of a column with one or two loads that 16 lanes
// make contiguous: one row (NT = 1), rows 2 i and 2 i + 1 of the first 32
// (NT = 2, 3, and 4 for FP64), row 32 + i (NT = 3), rows 32 + 2 i .. (NT = 4,
// FP64) or rows 4 i .. 4 i + 3 at once (NT = 4).  fwd2x_row names the row
// that tile t takes from lane i.  Lanes whose rows lie past ld read the
// column's last rows again, into rows of the result that are not stored.
// Bound by HBM and by the z rows that every column reads from L2 (64 or 128
// bytes against 160 or 320 of an FP32 or FP64 panel column of 40 rows):
// without the z reads it takes 85% of its time.  By the counters HBM moves 5.0
// (FP64), 4.5 (FP32) and 4.2 TB/s (FP16 factors), a third to a half of the
// requests hit L2, and the matrix cores are busy for a quarter to a third.  16
// columns at N = 81,920, FP64 1,102 -> 755 us, FP32 424 us; FP16 factors at N =
// 162,000 911 -> 630 us.  One to four batches in flight, 1,024- or 4,096-column
// units and 1,024 to 8,192 workgroups give the same within 5%.
template <typename E, int NT>
__device__ inline int fwd2x_row(int t, int i) {
  if (NT == 1) return i;
  if (NT == 4 && sizeof(E) < 8) return 4 * i + t;
  if (t < 2) return 2 * i + t;
  return NT == 3 ? 32 + i : 32 + 2 * i + (t - 2);
}

// KQ quads of columns with their z rows, read straight from memory.
template <typename E, typename A, int NR, int KQ, int NT>
struct ColBatch {
  E av[KQ][NT];
  A bv[KQ];
  // columns c0 + 4 u + lq; mc: the map entries of the batch (lane = column),
  // or, without a map, the z row of column 0; r1, r2: the lane's first rows
  template <bool MAP>
  __device__ inline void load(const E* __restrict__ P, const A* __restrict__ z, int mc, int c0,
                              int w, int ld, int r1, int r2, int xo, int lq) {
#pragma unroll
    for (int u = 0; u < KQ; ++u) {
      const int zi = MAP ? __shfl(mc, 4 * u + lq, 64) : mc + min(c0 + 4 * u + lq, w - 1);
      const uint32_t pc = (uint32_t)(min(c0 + 4 * u + lq, w - 1) * ld);   // 32 bits hold a unit
      if constexpr (NT == 4 && sizeof(E) < 8) {
        load_n<E, 4, true>(at32(P, pc + r1), av[u]);
      } else {
        load_n<E, NT == 1 ? 1 : 2, true>(at32(P, pc + r1), av[u]);
        if constexpr (NT >= 3) load_n<E, NT - 2, true>(at32(P, pc + r2), av[u] + 2);
      }
      bv[u] = z[(int64_t)zi * NR + xo];
    }
  }
  // only the columns below w
  __device__ inline void mask(int c0, int w, int lq) {
#pragma unroll
    for (int u = 0; u < KQ; ++u) {
      const bool ok = c0 + 4 * u + lq < w;
      bv[u] = ok ? bv[u] : (A)0;
#pragma unroll
      for (int t = 0; t < NT; ++t) av[u][t] = ok ? av[u][t] : (E)0;
    }
  }
  __device__ inline void mul(typename Mfma<A>::V (&acc)[NT]) {
#pragma unroll
    for (int u = 0; u < KQ; ++u)
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[t] = mfma16((A)av[u][t], bv[u], acc[t]);
  }
};

// The columns of a unit for one wavefront: batches of 4 KQ columns round-robin
// over the four wavefronts, two in turn, so that the next batch's loads are
// in flight while the current one is multiplied.  The column map (lane =
// column) runs two batches ahead and is read before the panel loads of its
// iteration, so that waiting for it waits for nothing newer; loads past the
// end are clamped, not skipped, so that no branch makes the waits
// conservative.  The last, partial batch of the unit goes after the loop.
template <typename E, typename A, int NR, int KQ, int NT>
__device__ inline void fwd2x_cols(const E* __restrict__ P, const int32_t* __restrict__ map,
                                  int w, int ld, const A* __restrict__ z, int wave, int lane,
                                  A (*ybuf)[NR]) {
  constexpr int CB = 4 * KQ, STEP = 4 * CB;
  const int lr = lane & 15, lq = lane >> 4;
  const int f1 = fwd2x_row<E, NT>(0, lr), f2 = NT >= 3 ? fwd2x_row<E, NT>(2, lr) : 0;
  // (clamped to the column's last rows: the same cache line as its neighbours)
  const int r1 = min(f1, ld - (NT == 1 ? 1 : (NT == 4 && sizeof(E) < 8 ? 4 : 2)));
  const int r2 = NT >= 3 ? min(f2, ld - (NT - 2)) : 0;
  const int xo = lr & (NR - 1);                 // NR = 8: columns 8 .. 15 repeat, not stored
  const int ml = lane & (CB - 1);
  typename Mfma<A>::V acc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[t] = typename Mfma<A>::V{0, 0, 0, 0};
  auto at = [&](int c) { return map[min(c + ml, w - 1)]; };
  ColBatch<E, A, NR, KQ, NT> b0, b1;
  int c = wave * CB;
  if (c + CB <= w) {
    int ma = at(c), mb = at(c + STEP);
    b0.template load<true>(P, z, ma, c, w, ld, r1, r2, xo, lq);
    for (; c + STEP + CB <= w; c += 2 * STEP) {         // two batches, no branch between them
      ma = at(c + 2 * STEP);
      b1.template load<true>(P, z, mb, c + STEP, w, ld, r1, r2, xo, lq);
      __builtin_amdgcn_sched_barrier(0);
      b0.mul(acc);
      mb = at(c + 3 * STEP);
      b0.template load<true>(P, z, ma, c + 2 * STEP, w, ld, r1, r2, xo, lq);
      __builtin_amdgcn_sched_barrier(0);
      b1.mul(acc);
    }
    if (c + CB <= w) {
      b0.mul(acc);
      c += STEP;
    }
  }
  if (c < w) {
    b0.template load<true>(P, z, at(c), c, w, ld, r1, r2, xo, lq);
    b0.mask(c, w, lq);
    b0.mul(acc);
  }
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (lr < NR) ybuf[fwd2x_row<E, NT>(t, Mfma<A>::row(j, lq))][lr] = acc[t][j];
}

template <typename E, typename A, int NR>
__device__ inline void fwd2x_unit(const E* __restrict__ P, const int32_t* __restrict__ map, int w,
                                  int ld, const A* __restrict__ z, int wave, int lane,
                                  A (*ybuf)[NR]) {
  constexpr int KQ = sizeof(A) == 8 ? 2 : 4;
  switch ((ld + 15) / 16) {                             // uniform over the workgroup
    case 1: fwd2x_cols<E, A, NR, KQ, 1>(P, map, w, ld, z, wave, lane, ybuf); break;
    case 2: fwd2x_cols<E, A, NR, KQ, 2>(P, map, w, ld, z, wave, lane, ybuf); break;
    case 3: fwd2x_cols<E, A, NR, KQ, 3>(P, map, w, ld, z, wave, lane, ybuf); break;
    default: fwd2x_cols<E, A, NR, KQ, 4>(P, map, w, ld, z, wave, lane, ybuf); break;
  }
}

// One workgroup per work unit; the four wavefronts' sums are added in LDS in
// a fixed order.
template <typename TD, typename TL, typename A, int NR>
__global__ __launch_bounds__(256) void k_fwd2x(const Unit* __restrict__ units, int64_t nunits,
                                               const int32_t* __restrict__ colmap,
                                               const A* __restrict__ z,
                                               A* __restrict__ ypart, int ldmax) {
  static_assert(NR == 8 || NR == 16, "MFMA phase 2 takes 8 or 16 right-hand sides");
  __shared__ A ybuf[4][kMaxLeaf][NR];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t per = (nunits + kXcds - 1) / kXcds;
  for (int64_t li = blockIdx.x; li < per * kXcds; li += gridDim.x) {
    const int64_t u = xcd_item(li, per);
    if (u >= nunits) continue;                          // uniform over the workgroup
    const Unit U = units[u];
    const int32_t* map = colmap + U.col;
    if (std::is_same<TD, TL>::value || U.dense)
      fwd2x_unit<TD, A, NR>(reinterpret_cast<const TD*>((uintptr_t)U.data), map, U.w, U.ld, z,
                            wave, lane, ybuf[wave]);
    else
      fwd2x_unit<TL, A, NR>(reinterpret_cast<const TL*>((uintptr_t)U.data), map, U.w, U.ld, z,
                            wave, lane, ybuf[wave]);
    const int m = U.m;
    __syncthreads();
    A* yp = ypart + u * ldmax * NR;
    for (int e = threadIdx.x; e < m * NR; e += blockDim.x) {
      const int row = e / NR, k = e % NR;
      yp[e] = ((ybuf[0][row][k] + ybuf[1][row][k]) + ybuf[2][row][k]) + ybuf[3][row][k];
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------------ transposed, phase 1
// Per row leaf: w[col0 + j] = sum_i P[i][j] x_c[i] for every panel column.
//
// Lane (cg, g) forms the partial dot of its granule of column group
// cg with x; the R partials of a column are then added by one lane, which
// reads them from the wavefront's own LDS area (a shift-down tree over the
// R lanes cost about four times the instructions per column).  Only the
// wavefront itself reads what it wrote: program order of its LDS
// instructions is enough, and wave_order keeps the compiler from
// moving LDS accesses across the exchange.
template <int NR>
constexpr int tr1_unr() { return NR <= 2 ? 4 : 1; }   // column groups per wavefront in flight

template <typename T, typename A, int NR, int G>
__device__ inline void tr1_run(const Unit& U, int ld, int R, int C, int cg, int g,
                               bool act, int wave, const A (&xg)[G][NR], A* __restrict__ w,
                               A* __restrict__ red) {
  static_assert(Gran<T>::G == G, "panel granules must cover the same rows");
  constexpr int UNR = tr1_unr<NR>();
  const int lane = threadIdx.x & 63;
  const int uw = U.w;
  const T* S = reinterpret_cast<const T*>((uintptr_t)U.data) + g * G;
  const int64_t col0 = U.col;
  const int ngrp = (uw + C - 1) / C;
  // a step covers the UNR C consecutive columns q0 C ... (q0 + UNR) C - 1;
  // reader t of a step sums column q0 C + t: group u = t / C, segment c
  const int ncol = UNR * C;
  const int ur = lane / C, cr = lane - ur * C;       // the reader's column in the first 64
  for (int q0 = wave * UNR; q0 < ngrp; q0 += 4 * UNR) {
    // UNR consecutive column groups, all granules loaded before any is reduced
    typename Gran<T>::E sv[UNR][G];
    bool ok[UNR];
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const int j = (q0 + u) * C + cg;
      ok[u] = act && q0 + u < ngrp && j < uw;
      Gran<T>::load(S + (int64_t)(ok[u] ? j : uw - 1) * ld, sv[u]);
    }
    // (without this the compiler may wait for one load before it issues the
    // next: 148 leaves of 23 to 45 rows, FP32, the kernel 26.3 us; 22 with it)
    __builtin_amdgcn_sched_barrier(0);
    A ps[UNR][NR];
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
#pragma unroll
      for (int k = 0; k < NR; ++k) ps[u][k] = 0;
#pragma unroll
      for (int e = 0; e < G; ++e) {
        const A x = ok[u] ? (A)sv[u][e] : (A)0;
#pragma unroll
        for (int k = 0; k < NR; ++k) ps[u][k] += x * xg[e][k];
      }
    }
    wave_order();                                   // the last step's reads are done
#pragma unroll
    for (int u = 0; u < UNR; ++u)
#pragma unroll
      for (int k = 0; k < NR; ++k) red[(u * 64 + lane) * NR + k] = ps[u][k];
    wave_order();
    for (int t = lane; t < ncol; t += 64) {
      int u = ur, c = cr;
      if (t >= 64) {
        u = t / C;
        c = t - u * C;
      }
      const A* rp = red + (u * 64 + c * R) * NR;
      A v[NR];
#pragma unroll
      for (int k = 0; k < NR; ++k) v[k] = 0;
      // partials added in order of g, read four at a time
      int e = 0;
      for (; e + 4 <= R; e += 4) {
        A r4[4][NR];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int k = 0; k < NR; ++k) r4[i][k] = rp[(e + i) * NR + k];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int k = 0; k < NR; ++k) v[k] += r4[i][k];
      }
      for (; e < R; ++e)
#pragma unroll
        for (int k = 0; k < NR; ++k) v[k] += rp[e * NR + k];
      const int jj = q0 * C + t;
      if (jj < uw) {
#pragma unroll
        for (int k = 0; k < NR; ++k) w[(col0 + jj) * NR + k] = v[k];
      }
    }
  }
}

template <typename TD, typename TL, typename A, int NR>
__global__ __launch_bounds__(256) void k_tr1(const Unit* __restrict__ units, int64_t nunits,
                                             const A* __restrict__ z, A* __restrict__ w) {
  constexpr int G = Gran<TD>::G;
  __shared__ A red[4][tr1_unr<NR>() * 64 * NR];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t per = (nunits + kXcds - 1) / kXcds;
  for (int64_t li = blockIdx.x; li < per * kXcds; li += gridDim.x) {
    const int64_t u = xcd_item(li, per);
    if (u >= nunits) continue;
    const Unit U = units[u];
    const int ld = U.ld, m = U.m, lo = U.lo;
    const int R = ld / G, C = 64 / R;
    const int cg = lane / R, g = lane % R;
    const bool act = cg < C;
    A xg[G][NR];
#pragma unroll
    for (int e = 0; e < G; ++e) {
      const int row = g * G + e;
#pragma unroll
      for (int k = 0; k < NR; ++k)
        xg[e][k] = (act && row < m) ? z[(int64_t)(lo + row) * NR + k] : (A)0;
    }
    if (std::is_same<TD, TL>::value || U.dense)
      tr1_run<TD, A, NR, G>(U, ld, R, C, cg, g, act, wave, xg, w, red[wave]);
    else
      tr1_run<TL, A, NR, G>(U, ld, R, C, cg, g, act, wave, xg, w, red[wave]);
  }
}

// The same on the matrix cores, for 4 to 16 right-hand sides and for small
// trees (see tr_mfma): the columns of a unit, 64 at a time per
// wavefront, are the terms of phase 1 (one leaf, the panel in place of the V
// slice).  On the vector units every column cost its own reduction over the
// rows.  Whole products at N = 32,000, leaf 64: FP64 4 columns 1,107 -> 447 us,
// 8 2,222 -> 509, 16 5,196 -> 686; FP32 4 columns 288 -> 247, 16 1,055 -> 395
// (leaf 32, 4 columns: 235 and 238; see tr_vec4_leaves).  Bound by HBM and by w
// itself, which is as many bytes as 2/5 of an FP32 panel of 40 rows at 16
// columns: N = 81,920, 5.7 (FP64), 4.9 (FP32) and 4.6 TB/s (FP16 factors), a
// quarter to a third of it written.
template <typename T, typename A, int NR>
__device__ inline void tr1x_unit(const Unit& U, const A* __restrict__ xt, A* __restrict__ w,
                                 int wave, int lane) {
  using V = typename Mfma<A>::V;
  const int lr = lane & 15, lq = lane >> 4;
  const int xo = lr & (NR - 1), ld = U.ld;
  const T* S = reinterpret_cast<const T*>((uintptr_t)U.data);
  const A* xb = xt + (int64_t)U.ldp * NR;
  for (int c0 = wave * 64; c0 < U.w; c0 += 256) {
    const int r = min(64, U.w - c0), ntile = (r + 15) / 16;
    V acc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = V{0, 0, 0, 0};
    const T* Sc = S + (int64_t)c0 * ld;
    auto go = [&](auto nt) {
      constexpr int NTL = decltype(nt)::value;
      int tc[NTL];
#pragma unroll
      for (int t = 0; t < NTL; ++t) tc[t] = min(t * 16 + lr, r - 1);
      fwd1x_leaf<T, A, NTL>(Sc, xb, ld, tc, xo, lq, acc);
    };
    switch (ntile) {                        // uniform over the wavefront
      case 1: go(std::integral_constant<int, 1>{}); break;
      case 2: go(std::integral_constant<int, 2>{}); break;
      case 3: go(std::integral_constant<int, 3>{}); break;
      default: go(std::integral_constant<int, 4>{}); break;
    }
#pragma unroll
    for (int t = 0; t < 4; ++t)
      if (t < ntile)
        tile_out<A, NR>(acc[t], lr, lq, [&](int row, int k, A v) {
          const int col = t * 16 + row;
          if (col < r) w[(U.col + c0 + col) * NR + k] = v;
        });
  }
}

template <typename TD, typename TL, typename A, int NR>
__global__ __launch_bounds__(256) void k_tr1x(const Unit* __restrict__ units, int64_t nunits,
                                              const A* __restrict__ xt, A* __restrict__ w) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t per = (nunits + kXcds - 1) / kXcds;
  for (int64_t li = blockIdx.x; li < per * kXcds; li += gridDim.x) {
    const int64_t u = xcd_item(li, per);
    if (u >= nunits) continue;
    const Unit U = units[u];
    if (std::is_same<TD, TL>::value || U.dense)
      tr1x_unit<TD, A, NR>(U, xt, w, wave, lane);
    else
      tr1x_unit<TL, A, NR>(U, xt, w, wave, lane);
  }
}

// s_b[l] = sum over the row leaves of b of w[ucol + l]  ->  z[n + toff + l].
// The sums of one block, lane = (group, term): with r <= 16 (32) the
// wavefront splits into four (two) groups of 16 (32) lanes; group g adds the
// row leaves q = g, g + groups, ... and the groups are added by shifts at
// the end.  Ranks above 64 take their terms 64 at a time.
template <typename A, int NR>
__device__ inline void tr_sums_block(const LrMeta& M, const int64_t* __restrict__ ucol,
                                     const A* __restrict__ w, A* __restrict__ z, int64_t n,
                                     const float* __restrict__ su, int lane) {
  const int nk = M.nt;
  const int gw = M.r <= 16 ? 16 : (M.r <= 32 ? 32 : 64);   // uniform over the wavefront
  const int ng = 64 / gw, grp = lane / gw;
  for (int t0 = 0; t0 < M.r; t0 += 64) {
    const int l = t0 + lane % gw;
    const bool ok = l < M.r;
    A acc[NR];
#pragma unroll
    for (int k = 0; k < NR; ++k) acc[k] = 0;
    if (ok) {
      // four row leaves per step with their loads in flight together
      int q = grp;
      for (; q + 3 * ng < nk; q += 4 * ng) {
        A v[4][NR];
#pragma unroll
        for (int u = 0; u < 4; ++u)
          load_row<A, NR>(w + (ucol[M.ub + q + u * ng] + l) * NR, v[u]);
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int k = 0; k < NR; ++k) acc[k] += v[u][k];
      }
      for (; q < nk; q += ng) {
        const int64_t col = ucol[M.ub + q] + l;
#pragma unroll
        for (int k = 0; k < NR; ++k) acc[k] += w[col * NR + k];
      }
    }
    for (int sh = gw; sh < 64; sh <<= 1) {
#pragma unroll
      for (int k = 0; k < NR; ++k) {
        const A o = __shfl_down(acc[k], sh, 64);
        acc[k] += o;
      }
    }
    if (grp == 0 && ok) {
      const A sc = su ? (A)su[M.toff + l] : (A)1;
#pragma unroll
      for (int k = 0; k < NR; ++k) z[(n + M.toff + l) * NR + k] = acc[k] * sc;
    }
  }
}

// One wavefront per four consecutive blocks.  When all four have rank <= 16
// (most blocks: the small ones), each 16-lane group takes one block and adds
// its row leaves in order, so the four dependent chains (descriptor, column
// offsets, sums, store) overlap; otherwise the wavefront takes the four
// blocks one after another as above.
template <typename A, int NR>
__global__ __launch_bounds__(256) void k_tr_sums(const LrMeta* __restrict__ meta, int64_t nl,
                                                 const int64_t* __restrict__ ucol,
                                                 const A* __restrict__ w, A* __restrict__ z,
                                                 int64_t n, const float* __restrict__ su) {
  const int lane = threadIdx.x & 63;
  const int64_t wid = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t nw = (int64_t)gridDim.x * 4;
  const int64_t nq = (nl + 3) / 4;
  const int grp = lane >> 4, l = lane & 15;
  for (int64_t qd = wid; qd < nq; qd += nw) {
    const int64_t b = qd * 4 + grp;
    const bool has = b < nl;
    const LrMeta M = meta[has ? b : nl - 1];
    if (__all(!has || M.r <= 16)) {                     // uniform over the wavefront
      if (has && l < M.r) {
        const int nk = M.nt;
        A acc[NR];
#pragma unroll
        for (int k = 0; k < NR; ++k) acc[k] = 0;
        for (int q = 0; q < nk; ++q) {
          const int64_t col = ucol[M.ub + q] + l;
#pragma unroll
          for (int k = 0; k < NR; ++k) acc[k] += w[col * NR + k];
        }
        const A sc = su ? (A)su[M.toff + l] : (A)1;
#pragma unroll
        for (int k = 0; k < NR; ++k) z[(n + M.toff + l) * NR + k] = acc[k] * sc;
      }
    } else {
      for (int g = 0; g < 4; ++g) {
        const int64_t bg = qd * 4 + g;
        if (bg < nl) tr_sums_block<A, NR>(meta[bg], ucol, w, z, n, su, lane);
      }
    }
  }
}

// ------------------------------------------------------------------ transposed, phase 2
// Per column leaf: dense blocks contribute w entries (kind 0, lane = output
// row), V slices contribute V s (kind 1, granule product).  The items of a
// leaf are dealt to S workgroups (item i to workgroup (i / 4) mod S, wavefront
// i mod 4), so that a leaf's few hundred slices are not one long chain of
// dependent loads per wavefront; with S > 1 each workgroup writes its partial
// rows to ypart[c S + s] and k_tr2_sum adds them in order of s.
// The columns of a V item go up to UMAX groups of C at a time, by what is left
// of it: with four at a time whatever the width, trees of narrow items (blocks
// that stand alone, 9.5 columns) paid for loads of nothing: N = 200,000, FP32,
// leaf 24, one and two columns 2,450 and 3,050 us, with one at a time 2,150 and
// 2,400.  Wide items want the loads in flight (N = 32,000, leaf 32 and 64, FP32
// 183 -> 174 and 190 -> 185, FP16 129 -> 121 and 150 -> 142 against one at a
// time), unless their sums take too many registers: two for two double columns
// of float or half slices (N = 81,920, leaf 32: FP32 814 -> 799, FP16 530 -> 503
// us), one for four columns (62 registers, 86 with four: N = 162,000, leaf 24,
// 1,709 and 1,844 us).
template <typename T, typename A, int NR>
constexpr int tr2_groups() {
  return NR >= 4 ? 1 : (sizeof(A) == 8 && sizeof(T) < 8 && NR == 2 ? 2 : 4);
}
template <typename T, typename A, typename VT, int NR, int UMAX>
__global__ __launch_bounds__(256) void k_tr2(const int32_t* __restrict__ beg,
                                             const TItem* __restrict__ items, MvLeaves L,
                                             const A* __restrict__ w, const A* __restrict__ z,
                                             int64_t n, const int32_t* __restrict__ perm,
                                             VT* __restrict__ y, int nrhs, int k0, int nv, int S,
                                             A* __restrict__ ypart, int ldmax) {
  constexpr int G = Gran<T>::G;
  __shared__ A ybuf[4][kMaxLeaf][NR];
  // wave-uniform index: item descriptors come in by scalar loads
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t nwork = L.nleaf * S;
  const int64_t per = (nwork + kXcds - 1) / kXcds;
  for (int64_t li = blockIdx.x; li < per * kXcds; li += gridDim.x) {
    const int64_t q = xcd_item(li, per);
    if (q >= nwork) continue;                           // uniform over the workgroup
    const int64_t c = q / S;
    const int sp = (int)(q - c * S);
    const int ld = (int)(L.ldpre[c + 1] - L.ldpre[c]);
    const int R = ld / G, C = 64 / R;
    const int cg = lane / R, g = lane % R;
    const bool act = cg < C;
    const int m = L.m[c], lo = L.lo[c];
    A acc[G][NR], yT[NR];
#pragma unroll
    for (int k = 0; k < NR; ++k) {
      yT[k] = 0;
#pragma unroll
      for (int e = 0; e < G; ++e) acc[e][k] = 0;
    }
    const int b0 = beg[c], b1 = beg[c + 1];
    // the next item's descriptor is loaded one iteration ahead
    const int it0 = b0 + 4 * sp + wave;
    TItem In;
    if (it0 < b1) In = items[it0];
    for (int it = it0; it < b1; it += 4 * S) {
      const TItem I = In;
      if (it + 4 * S < b1) In = items[it + 4 * S];
      if (I.kind == 0) {
        if (lane < I.w) {
#pragma unroll
          for (int k = 0; k < NR; ++k) yT[k] += w[(I.src + lane) * NR + k];
        }
      } else {
        const T* S = reinterpret_cast<const T*>((uintptr_t)I.data);
        // U column groups with unconditional loads (a lane without a column
        // reads the slice's last one and adds zero), so that all their loads
        // are in flight together
        auto groups = [&](auto cnt, int j0) {
          constexpr int U = decltype(cnt)::value;
          typename Gran<T>::E s[U][G];
          A zz[U][NR];
          bool ok[U];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int j = j0 + u * C + cg;
            ok[u] = act && j < I.w;
            const int jj = ok[u] ? j : I.w - 1;
            Gran<T>::load(S + (int64_t)jj * ld + g * G, s[u]);
            load_row<A, NR>(z + (n + I.src + jj) * NR, zz[u]);
          }
          __builtin_amdgcn_sched_barrier(0);            // all loads before the first wait
#pragma unroll
          for (int u = 0; u < U; ++u)
#pragma unroll
            for (int e = 0; e < G; ++e)
#pragma unroll
              for (int k = 0; k < NR; ++k)
                acc[e][k] += (A)s[u][e] * (ok[u] ? zz[u][k] : (A)0);
        };
        for (int j0 = 0; j0 < I.w;) {                   // uniform over the wavefront
          const int left = I.w - j0;
          if (UMAX == 4 && left > 2 * C) {
            groups(std::integral_constant<int, 4>{}, j0);
            j0 += 4 * C;
          } else if (UMAX >= 2 && left > C) {
            groups(std::integral_constant<int, 2>{}, j0);
            j0 += 2 * C;
          } else {
            const int j = j0 + cg;
            if (act && j < I.w) {
              typename Gran<T>::E s[G];
              Gran<T>::load(S + (int64_t)j * ld + g * G, s);
              A zz[NR];
              load_row<A, NR>(z + (n + I.src + j) * NR, zz);
#pragma unroll
              for (int e = 0; e < G; ++e)
#pragma unroll
                for (int k = 0; k < NR; ++k) acc[e][k] += (A)s[e] * zz[k];
            }
            j0 += C;
          }
        }
      }
    }
#pragma unroll
    for (int e = 0; e < G; ++e)
#pragma unroll
      for (int k = 0; k < NR; ++k) {
        A v = acc[e][k];
        for (int s = 1; s < C; s <<= 1) {
          const A o = __shfl_down(v, s * R, 64);
          if (cg + s < C) v += o;
        }
        acc[e][k] = v;
      }
    if (cg == 0) {
#pragma unroll
      for (int e = 0; e < G; ++e) {
        const int row = g * G + e;
        if (row < kMaxLeaf)
#pragma unroll
          for (int k = 0; k < NR; ++k) ybuf[wave][row][k] = acc[e][k];
      }
    }
    __syncthreads();
    if (lane < m) {
#pragma unroll
      for (int k = 0; k < NR; ++k) ybuf[wave][lane][k] += yT[k];
    }
    __syncthreads();
    A* yp = ypart + q * ldmax * NR;
    for (int e = threadIdx.x; e < m * NR; e += blockDim.x) {
      const int row = e / NR, k = e % NR;
      const A v = ((ybuf[0][row][k] + ybuf[1][row][k]) + ybuf[2][row][k]) + ybuf[3][row][k];
      if (S > 1)
        yp[e] = v;
      else if (k < nv)
        y[(int64_t)perm[lo + row] * nrhs + k0 + k] = (VT)v;
    }
    __syncthreads();
  }
}

// The same on the matrix cores, where phase 1 runs there: V items are
// column batches as in the forward phase 2, with consecutive z rows; the w
// entries of dense items, NR values per row of the leaf, are read as one
// contiguous run, value e by lane e mod 64.  Bound by latency: wavefronts wait
// 80% of their time, and HBM moves 3.8 (FP64), 3.2 (FP32) and 2.5 TB/s (FP16)
// with 16 columns at N = 81,920 (729, 434 and 287 us): items are a descriptor,
// then one or two batches of loads.
template <typename T, typename A, int NR, int NT>
__device__ inline void tr2x_items(const TItem* __restrict__ items, int it0, int b1, int step,
                                  int ld, const A* __restrict__ w, const A* __restrict__ z,
                                  int64_t n, int lane, A (*ybuf)[NR]) {
  constexpr int KQ = sizeof(A) == 8 ? 2 : 4, CB = 4 * KQ;
  const int lr = lane & 15, lq = lane >> 4;
  const int f1 = fwd2x_row<T, NT>(0, lr), f2 = NT >= 3 ? fwd2x_row<T, NT>(2, lr) : 0;
  const int r1 = min(f1, ld - (NT == 1 ? 1 : (NT == 4 && sizeof(T) < 8 ? 4 : 2)));
  const int r2 = NT >= 3 ? min(f2, ld - (NT - 2)) : 0;
  const int xo = lr & (NR - 1);
  typename Mfma<A>::V acc[NT];
  A yd[NR];                                     // dense items: values lane + 64 k of rows x NR
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[t] = typename Mfma<A>::V{0, 0, 0, 0};
#pragma unroll
  for (int k = 0; k < NR; ++k) yd[k] = 0;
  TItem In;
  if (it0 < b1) In = items[it0];
  for (int it = it0; it < b1; it += step) {
    const TItem I = In;
    if (it + step < b1) In = items[it + step];          // one iteration ahead
    if (I.kind == 0) {
      const A* ws = w + I.src * NR;
#pragma unroll
      for (int k = 0; k < NR; ++k)
        if (lane + 64 * k < I.w * NR) yd[k] += ws[lane + 64 * k];
    } else {
      const T* P = reinterpret_cast<const T*>((uintptr_t)I.data);
      const A* zb = z + (n + I.src) * NR;
      ColBatch<T, A, NR, KQ, NT> b0, b1b;
      // two batches at a time, and one for what is left of narrow items
      int c = 0;
      for (; c + CB < I.w; c += 2 * CB) {               // uniform over the wavefront
        b0.template load<false>(P, zb, 0, c, I.w, ld, r1, r2, xo, lq);
        b1b.template load<false>(P, zb, 0, c + CB, I.w, ld, r1, r2, xo, lq);
        if (c + 2 * CB > I.w) b1b.mask(c + CB, I.w, lq);
        b0.mul(acc);
        b1b.mul(acc);
      }
      if (c < I.w) {
        b0.template load<false>(P, zb, 0, c, I.w, ld, r1, r2, xo, lq);
        b0.mask(c, I.w, lq);
        b0.mul(acc);
      }
    }
  }
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (lr < NR) ybuf[fwd2x_row<T, NT>(t, Mfma<A>::row(j, lq))][lr] = acc[t][j];
  wave_order();
  A* yf = &ybuf[0][0];
#pragma unroll
  for (int k = 0; k < NR; ++k)                          // 64 NR values, rows past the tiles unused
    if (lane + 64 * k < NT * 16 * NR) yf[lane + 64 * k] += yd[k];
}

template <typename T, typename A, typename VT, int NR>
__global__ __launch_bounds__(256) void k_tr2x(const int32_t* __restrict__ beg,
                                              const TItem* __restrict__ items, MvLeaves L,
                                              const A* __restrict__ w, const A* __restrict__ z,
                                              int64_t n, const int32_t* __restrict__ perm,
                                              VT* __restrict__ y, int nrhs, int k0, int nv, int S,
                                              A* __restrict__ ypart, int ldmax) {
  __shared__ A ybuf[4][kMaxLeaf][NR];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t nwork = L.nleaf * S;
  const int64_t per = (nwork + kXcds - 1) / kXcds;
  for (int64_t li = blockIdx.x; li < per * kXcds; li += gridDim.x) {
    const int64_t q = xcd_item(li, per);
    if (q >= nwork) continue;                           // uniform over the workgroup
    const int64_t c = q / S;
    const int sp = (int)(q - c * S);
    const int ld = (int)(L.ldpre[c + 1] - L.ldpre[c]);
    const int m = L.m[c], lo = L.lo[c];
    const int it0 = beg[c] + 4 * sp + wave, b1 = beg[c + 1];
    switch ((ld + 15) / 16) {                           // uniform over the workgroup
      case 1: tr2x_items<T, A, NR, 1>(items, it0, b1, 4 * S, ld, w, z, n, lane, ybuf[wave]); break;
      case 2: tr2x_items<T, A, NR, 2>(items, it0, b1, 4 * S, ld, w, z, n, lane, ybuf[wave]); break;
      case 3: tr2x_items<T, A, NR, 3>(items, it0, b1, 4 * S, ld, w, z, n, lane, ybuf[wave]); break;
      default: tr2x_items<T, A, NR, 4>(items, it0, b1, 4 * S, ld, w, z, n, lane, ybuf[wave]); break;
    }
    __syncthreads();
    A* yp = ypart + q * ldmax * NR;
    for (int e = threadIdx.x; e < m * NR; e += blockDim.x) {
      const int row = e / NR, k = e % NR;
      const A v = ((ybuf[0][row][k] + ybuf[1][row][k]) + ybuf[2][row][k]) + ybuf[3][row][k];
      if (S > 1)
        yp[e] = v;
      else if (k < nv)
        y[(int64_t)perm[lo + row] * nrhs + k0 + k] = (VT)v;
    }
    __syncthreads();
  }
}

// y rows of every column leaf = sum of its S partial rows (in order of s),
// scattered to application order.
template <typename A, typename VT, int NR>
__global__ __launch_bounds__(256) void k_tr2_sum(MvLeaves L, int S, const A* __restrict__ ypart,
                                                 int ldmax, const int32_t* __restrict__ perm,
                                                 VT* __restrict__ y, int nrhs, int k0, int nv) {
  constexpr int LW = sum_leaves<NR>(), TL = 256 / LW;
  for (int64_t c = blockIdx.x * LW + threadIdx.x / TL; c < L.nleaf; c += (int64_t)gridDim.x * LW) {
    const int m = L.m[c], lo = L.lo[c];
    const A* yp = ypart + c * S * ldmax * NR;
    for (int e = threadIdx.x % TL; e < m * NR; e += TL) {
      const int row = e / NR, k = e % NR;
      A v = 0;
      for (int sp = 0; sp < S; ++sp) v += yp[(int64_t)sp * ldmax * NR + e];
      if (k < nv) y[(int64_t)perm[lo + row] * nrhs + k0 + k] = (VT)v;
    }
  }
}

// ------------------------------------------------------------------ host side
// Transposed products of one or two columns run on the matrix cores up to 128
// leaves (FP64 factors, or two columns in single precision) or 64, on the vector
// units above.  Small products wait for loads, and the matrix kernels have all
// the loads of 64 columns in flight; large ones are bound by HBM, where the
// vector kernels use fewer, longer wavefronts.  One and two columns, vector ->
// matrix: 64 leaves of 53 rows, FP64 63 -> 41 and 70 -> 44 us, FP32 37 -> 30 and
// 41 -> 33; 128 leaves of 45 rows, FP64 74 -> 53 and 79 -> 59, FP32 37 -> 39 and
// 43 -> 43, FP16 37 -> 37 and 42 -> 40, of 62 rows, FP32 45 -> 52 and 56 -> 57;
// 256 leaves of 45 rows, FP64 116 -> 123 and 132 -> 138, FP32 65 -> 69 and 73 ->
// 71; N = 81,920, leaf 64, FP32 532 -> 628 and 590 -> 666.
// FP32 factors with double vectors: 64 leaves of 53 rows 38 -> 37 and 45 -> 40,
// 128 leaves of 45 rows 42 -> 47 and 48 -> 50 us.  These (and FP16 factors,
// alike) go there from 2,200 elements on, or up to 16 leaves per column: 500
// elements, 8 leaves 21.0 -> 19.3 and 23.9 -> 21.9 us, 16 leaves the same; 1,280,
// 32 leaves 22.5 -> 25.0 and 26.6 -> 26.3, 64 leaves 22.0 -> 25.4 and 24.3 ->
// 25.3; 2,000, 64 leaves 26.3 -> 27.6 and 28.4 -> 28.1; 2,420, 64 leaves 31.5 ->
// 30.0 and 36.5 -> 32.5.
template <typename TL, typename A, int NR>
static bool tr_mfma(int64_t nleaf, int64_t n) {
  if (NR >= 4) return true;
  if (sizeof(TL) < 8 && sizeof(A) == 8) return nleaf <= 16 * NR || (nleaf <= 64 && n >= 2200);
  return nleaf <= (sizeof(TL) == 8 || NR == 2 ? 128 : 64);
}

// Four single-precision columns run on the vector units from this many leaves
// on (vcols: mean columns of a V item).  Blocks whose column leaves differ in ld
// stand alone, and their items are as wide as their rank: a quarter of a pass
// of the matrix kernel.  N = 200,000, 16,384 leaves of 12.2 rows (ld 12 and 16,
// 9.5 columns) 3,859 -> 2,824 us; N = 50,000, 1,024 leaves of 48.8 rows, 485 ->
// 438, 4,096 of 12.2, 661 -> 514, FP16 factors 359 -> 335 and 472 -> 397.  FP32
// with wide items: 2,048 leaves of 19.8 rows 387 -> 344, of 40 rows 722 -> 682,
// 4,096 of 39.6 rows 1,562 -> 1,509; fewer leaves 1,024 of 20 rows 171 and 169,
// of 39.6 rows 326 and 321, 512 of 22.5 rows 82 and 102.  FP16 with wide items:
// 2,048 leaves of 10 rows 167 and 202, of 40 rows 486 and 475, 4,096 of 39.6
// rows 983 and 1,043.
template <typename TL>
constexpr int64_t tr_vec4_leaves(double vcols) {
  return vcols < 24.0 ? 1024 : (sizeof(TL) == 4 ? 2048 : INT64_MAX);
}

template <typename TD, typename TL, typename A, typename VT, int NR>
static void mv_chunk(const MvPlan& P, const VT* x, VT* y, int nrhs, int k0, int nv,
                     bool transposed, hipStream_t s) {
  A* z = static_cast<A*>(P.z);
  A* w = static_cast<A*>(P.w);
  MvProfile* pr = P.prof;
  if (pr) HM_HIP(hipEventRecord(pr->ev[0], s));
  constexpr bool kVec4 = NR == 4 && sizeof(A) == 4;
  // transposed, on the matrix cores
  const bool tmx = tr_mfma<TL, A, NR>(P.L.nleaf, P.n) &&
                   !(kVec4 && P.L.nleaf >= tr_vec4_leaves<TL>(P.vitem / P.ldmax));
  // x per leaf, NR columns of ld values each.  Transposed products on the matrix
  // cores keep it where the others keep x and t: they read no other x, and t is
  // written when it has been read.  Forward ones keep it at the end of the memory
  // of ypart, which phase 2 writes after phase 1 has read x.  Not at its start,
  // and no transposed one there: lines that every XCD has just read are slow to
  // write (32 leaves of 40 rows, FP64, two columns, transposed: the column kernel
  // 13.7 us with x at the start, 10.6 at the end, whose lines it doesn't reach;
  // 8 leaves of 62 rows, FP32, 16 columns, which it does, the product 24.6 us,
  // 22.7 with x in z)
  const int64_t xt_bytes = P.xt_rows * NR * (int64_t)sizeof(A);
  const bool xt_in_z = transposed && tmx && xt_bytes <= P.z_bytes;
  A* xt = xt_in_z ? z
                  : reinterpret_cast<A*>(static_cast<char*>(P.ypart) +
                                         ((P.ypart_bytes - xt_bytes) & ~(int64_t)255));
  if (NR >= 4 || (transposed && tmx))
    k_gather_x<VT, A, NR><<<(unsigned)std::min<int64_t>(P.L.nleaf, 1 << 20), 256, 0, s>>>(
        x, nrhs, k0, nv, P.perm, P.L, xt_in_z ? nullptr : z, xt);
  else
    k_gather<VT, A><<<grid_for(P.n * NR, 256, 4096), 256, 0, s>>>(x, nrhs, k0, NR, P.perm, P.n, z);
  HM_LAUNCH_CHECK();
  if (pr) HM_HIP(hipEventRecord(pr->ev[1], s));
  if (!transposed) {
    // phase 1 over its work units (column chunks of the V panels)
    const int64_t nu = NR >= 4 ? P.nux : P.nu1;
    const unsigned g1 = (unsigned)std::max<int64_t>(1, std::min<int64_t>(ceil_div(nu, 4), 1 << 20));
    if (nu > 0) {
      if constexpr (NR >= 4)
        k_fwd1x<TL, A, NR><<<g1, 256, 0, s>>>(P.metax, P.nux, P.L, xt, z, P.n, P.su);
      else
        k_fwd1<TL, A, NR><<<g1, 256, 0, s>>>(P.meta1, P.nu1, P.L, z, P.n, P.su);
      HM_LAUNCH_CHECK();
    }
    if (pr) {
      HM_HIP(hipEventRecord(pr->ev[2], s));
      HM_HIP(hipEventRecord(pr->ev[3], s));
    }
    const unsigned gu = (unsigned)std::min<int64_t>(ceil_div(P.nunits, kXcds) * kXcds, P.grid);
    if (P.nunits > 0) {
      if constexpr (NR == 8 || NR == 16)
        k_fwd2x<TD, TL, A, NR><<<gu, 256, 0, s>>>(P.units, P.nunits, P.colmap, z, static_cast<A*>(P.ypart),
                                                        P.ldmax);
      else
        k_fwd2<TD, TL, A, NR><<<gu, 256, 0, s>>>(P.units, P.nunits, P.colmap, z,
                                                 static_cast<A*>(P.ypart), P.ldmax);
      HM_LAUNCH_CHECK();
    }
    k_fwd2_sum<A, VT, NR><<<(unsigned)std::min<int64_t>(ceil_div(P.L.nleaf, sum_leaves<NR>()), P.grid), 256, 0, s>>>(
        P.L, P.ubeg, static_cast<const A*>(P.ypart), P.ldmax, P.perm, y, nrhs, k0,
        nv);
    HM_LAUNCH_CHECK();
  } else {
    if (P.nunits > 0) {
      const unsigned gu = (unsigned)std::min<int64_t>(ceil_div(P.nunits, kXcds) * kXcds, P.grid);
      if (tmx)
        k_tr1x<TD, TL, A, NR><<<gu, 256, 0, s>>>(P.units, P.nunits, xt, w);
      else if constexpr (NR < 4 || kVec4)
        k_tr1<TD, TL, A, NR><<<gu, 256, 0, s>>>(P.units, P.nunits, z, w);
      HM_LAUNCH_CHECK();
    }
    if (pr) HM_HIP(hipEventRecord(pr->ev[2], s));
    if (P.nlr > 0) {
      // four blocks per wavefront, four wavefronts per workgroup; blocks
      // come largest first and stay round-robin over the XCDs
      const unsigned gq =
          (unsigned)std::max<int64_t>(1, std::min<int64_t>(ceil_div(ceil_div(P.nlr, 4), 4), 1 << 20));
      k_tr_sums<A, NR><<<gq, 256, 0, s>>>(P.meta, P.nlr, P.ucol, w, z, P.n, P.su);
      HM_LAUNCH_CHECK();
    }
    if (pr) HM_HIP(hipEventRecord(pr->ev[3], s));
    // workgroups per column leaf: up to 8, as many as the unit workspace
    // holds partial rows (ldmax x NR) for
    const int64_t cap = P.ypart_bytes / ((int64_t)P.ldmax * NR * (int64_t)sizeof(A));
    const int S = (int)std::max<int64_t>(1, std::min<int64_t>(8, cap / std::max<int64_t>(1, P.L.nleaf)));
    // leaves carry similar work: the grid covers the XCD-ordered index range
    const unsigned gt = (unsigned)std::min<int64_t>(ceil_div(P.L.nleaf * S, kXcds) * kXcds, P.grid);
    if (tmx)
      k_tr2x<TL, A, VT, NR><<<gt, 256, 0, s>>>(P.tbeg, P.titems, P.L, w, z, P.n, P.perm, y, nrhs,
                                               k0, nv, S, static_cast<A*>(P.ypart), P.ldmax);
    else if constexpr (NR < 4 || kVec4) {
      auto tr2 = [&](auto u) {
        k_tr2<TL, A, VT, NR, decltype(u)::value><<<gt, 256, 0, s>>>(
            P.tbeg, P.titems, P.L, w, z, P.n, P.perm, y, nrhs, k0, nv, S, static_cast<A*>(P.ypart),
            P.ldmax);
      };
      constexpr int UMAX = tr2_groups<TL, A, NR>();
      // items of hardly more than one group: nothing to keep in flight
      if (UMAX == 1 || 2.0 * P.vitem <= 3.0 * 64 * Gran<TL>::G)
        tr2(std::integral_constant<int, 1>{});
      else
        tr2(std::integral_constant<int, UMAX>{});
    }
    HM_LAUNCH_CHECK();
    if (S > 1) {
      k_tr2_sum<A, VT, NR><<<(unsigned)std::min<int64_t>(ceil_div(P.L.nleaf, sum_leaves<NR>()), P.grid), 256, 0, s>>>(
          P.L, S, static_cast<const A*>(P.ypart), P.ldmax, P.perm, y, nrhs, k0,
        nv);
      HM_LAUNCH_CHECK();
    }
  }
  if (pr) {
    HM_HIP(hipEventRecord(pr->ev[4], s));
    HM_HIP(hipEventSynchronize(pr->ev[4]));
    const int base = transposed ? 4 : 0;
    for (int k = 0; k < 4; ++k) {
      float ms = 0.f;
      HM_HIP(hipEventElapsedTime(&ms, pr->ev[k], pr->ev[k + 1]));
      pr->ms[base + k] += ms;
      pr->launches[base + k] += 1;
    }
  }
}

// Columns of the next pass for `left` remaining ones: a pass reads the whole
// stored operator once whatever its width, so a wider pass with zero columns
// beats two narrow ones.
static int pass_width(int left, int cap) {
  int w = left >= 9 ? 16 : (left >= 5 ? 8 : (left >= 3 ? 4 : left));
  while (w > cap) w >>= 1;
  return w;
}

template <typename TD, typename TL, typename A, typename VT>
void matvec_impl(const MvPlan& P, const VT* x, VT* y, int nrhs, bool transposed, hipStream_t s) {
  const int cap = transposed ? P.max_nr_t : 16;
  for (int k0 = 0; k0 < nrhs;) {
    const int w = pass_width(nrhs - k0, cap), nv = std::min(w, nrhs - k0);
    switch (w) {
      case 16: mv_chunk<TD, TL, A, VT, 16>(P, x, y, nrhs, k0, nv, transposed, s); break;
      case 8: mv_chunk<TD, TL, A, VT, 8>(P, x, y, nrhs, k0, nv, transposed, s); break;
      case 4: mv_chunk<TD, TL, A, VT, 4>(P, x, y, nrhs, k0, nv, transposed, s); break;
      case 2: mv_chunk<TD, TL, A, VT, 2>(P, x, y, nrhs, k0, nv, transposed, s); break;
      default: mv_chunk<TD, TL, A, VT, 1>(P, x, y, nrhs, k0, nv, transposed, s); break;
    }
    k0 += nv;
  }
}

// storage 0: FP64, 1: FP32, 2: FP32 dense + FP16 factors.  Vectors VT;
// accumulation in double unless the storage and the vectors are single
// precision.
void matvec_dispatch(const MvPlan& P, int storage, const void* x, void* y, int nrhs, int vec_f32,
                     bool transposed, hipStream_t s) {
  if (storage == 2) {
    if (vec_f32)
      matvec_impl<float, _Float16, float, float>(P, (const float*)x, (float*)y, nrhs, transposed, s);
    else
      matvec_impl<float, _Float16, double, double>(P, (const double*)x, (double*)y, nrhs,
                                                    transposed, s);
  } else if (storage == 1) {
    if (vec_f32)
      matvec_impl<float, float, float, float>(P, (const float*)x, (float*)y, nrhs, transposed, s);
    else
      matvec_impl<float, float, double, double>(P, (const double*)x, (double*)y, nrhs, transposed,
                                                s);
  } else {
    if (vec_f32)
      matvec_impl<double, double, double, float>(P, (const float*)x, (float*)y, nrhs, transposed,
                                                 s);
    else
      matvec_impl<double, double, double, double>(P, (const double*)x, (double*)y, nrhs,
                                                  transposed, s);
  }
}

}  // namespace hm
