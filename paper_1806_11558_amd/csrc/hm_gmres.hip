// Vector kernels of the restarted GMRES solver (double precision Arnoldi).
//
// The paper solves its symmetric Galerkin system by CG with one H-matrix
// product per step (Sec. 4.1); the collocation matrix is not symmetric, so
// its solve is GMRES with the same product.  Both are here.  All reductions
// write per-tile partial sums that a second kernel adds in a fixed order, so
// the solve is bitwise reproducible.
#include <algorithm>

#include "hm_internal.h"
#include "hm_wave.h"

namespace hm {

// ------------------------------------------------------------------ Arnoldi step
// Classical Gram-Schmidt, twice, in three kernels after the product:
//   first   part = Q^T w                          (partial dots per row tile)
//   second  w' = w - Q h1, part = Q^T w'          (h1 = the sums of part)
//   last    w'' = w' - Q h2, part = |w''|^2       (h2 likewise)
//   next    q = w'' / |w''| into the basis and into the product's input, the
//           coefficients h1 + h2 and |w''| to the host
// A dot product needs the finished vector of its own rows only, so the update
// of one pass and the dots of the next share a kernel.  Before, a step was
// nine kernels, two copies and a synchronisation beside its product (40 of
// 130 us of kernels at N = 5,120); these are four and no copy.
//
// The rows are cut into tiles of gs_tile() rows: about 96 tiles, so that small
// systems still spread over the chip, and at most kGsElems elements each in
// one piece.  With few tiles (GsShape::fold) every workgroup adds the tile
// sums it needs itself, else gs_final adds them once per pass.
namespace {
constexpr int kGT = 256;
constexpr int kGsElems = 2048;     // elements of w held in LDS at a time
constexpr int kGsVecs = 16;        // basis vectors per workgroup of the dots
constexpr int kGsH = 512;          // coefficients held in LDS at a time
}  // namespace

GsShape gs_shape(int64_t n, int nr, bool coarse) {
  GsShape g;
  g.n = n;
  g.nr = nr;
  const int64_t tot = n * nr;
  int64_t et = (ceil_div(tot, 96) + 127) / 128 * 128;
  et = std::min<int64_t>(std::max<int64_t>(et, 128), kGsElems);
  g.tr = coarse ? kGsElems : std::max<int64_t>(1, et / nr);
  g.tiles = (int)ceil_div(n, g.tr);
  // Every workgroup adds all sums of a step: with many columns that takes
  // longer than the kernels saved (graph solve, N = 20, 24 columns: 1,330 us,
  // 1,160 as separate kernels).  (coarse: the second array of partial sums
  // that folding takes is left out)
  g.fold = !coarse && nr <= 16 && (int64_t)g.tiles * nr <= 160;
  g.coarse = coarse;
  return g;
}

// Sum over the tiles of partial sum e = k nr + c (part[e * tiles + t]); one
// wavefront, lanes over the tiles, a fixed order.
__device__ inline double gs_tile_sum(const double* __restrict__ part, int64_t e, int tiles) {
  double s = 0.0;
  for (int t = threadIdx.x & 63; t < tiles; t += 64) s += part[e * tiles + t];
  return wsum(s);
}

// Partial dots of the basis vectors [k0, k1) with the cnt elements of w held
// in LDS (they start at element e0 of every vector): one wavefront per vector
// and group of up to 64 columns.  A power of two of columns keeps every lane's
// column fixed (lane mod nr) with contiguous reads; any other count gives its
// columns to consecutive lanes, as many rows at once as fit (taken one by one,
// 40 columns at N = 80 cost 1.2 times the solve).  add: the tile's earlier
// pieces are there.
__device__ inline void gs_dots(const double* __restrict__ Q, int64_t ldq, int k0, int k1,
                               const double* __restrict__ ws, int64_t e0, int cnt, int nr,
                               int tiles, int tile, bool add, double* __restrict__ part) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const bool pow2 = nr <= 64 && (nr & (nr - 1)) == 0;
  const int nch = (nr + 63) / 64;
  for (int task = wave; task < (k1 - k0) * nch; task += kGT / 64) {
    const int k = k0 + task / nch, c0 = task % nch * 64, cw = min(64, nr - c0);
    const double* q = Q + (int64_t)k * ldq + e0;
    double acc = 0.0;
    if (pow2) {
#pragma unroll 4
      for (int e = lane; e < cnt; e += 64) acc += q[e] * ws[e];
      if (nr == 1) {
        acc = wsum(acc);
      } else {
        for (int off = 32; off >= nr; off >>= 1) acc += __shfl_xor(acc, off, 64);
      }
    } else {
      const int rows = 64 / cw, g = lane / cw;
      if (g < rows)
        for (int e = g * nr + c0 + (lane - g * cw); e < cnt; e += rows * nr) acc += q[e] * ws[e];
      for (int s = 1; s < rows; s <<= 1) {
        const double o = __shfl_down(acc, s * cw, 64);
        if (g + s < rows) acc += o;
      }
    }
    if (lane < cw) {
      double* o = part + ((int64_t)k * nr + c0 + lane) * tiles + tile;
      *o = add ? *o + acc : acc;
    }
  }
}

// j: the step, from the argument or, in a captured graph, from jd[0].
__device__ inline int gs_step(const int64_t* jd, int j) { return jd ? (int)jd[0] : j; }

template <typename W>
__global__ __launch_bounds__(kGT) void k_gs_first(const double* __restrict__ Q, int64_t ldq,
                                                  const int64_t* __restrict__ jd, int nk,
                                                  const W* __restrict__ w, GsShape G,
                                                  double* __restrict__ part) {
  __shared__ double ws[kGsElems];
  const int nv = jd ? (int)jd[0] + 1 : nk;
  const int k0 = blockIdx.y * kGsVecs, k1 = min(k0 + kGsVecs, nv);
  if (k0 >= nv) return;                                 // uniform over the workgroup
  const int64_t r0 = (int64_t)blockIdx.x * G.tr, r1 = min(r0 + G.tr, G.n);
  const int sr = kGsElems / G.nr;
  for (int64_t r = r0; r < r1; r += sr) {
    const int cnt = (int)min((int64_t)sr, r1 - r) * G.nr;
    const int64_t e0 = r * G.nr;
    __syncthreads();                                    // the previous piece is consumed
    for (int e = threadIdx.x; e < cnt; e += kGT) ws[e] = (double)w[e0 + e];
    __syncthreads();
    gs_dots(Q, ldq, k0, k1, ws, e0, cnt, G.nr, G.tiles, blockIdx.x, r > r0, part);
  }
}

// out = in - Q h for the tile, h the sums of part_in (fold) or hsum, then the
// partial dots Q^T out (LAST = false) or |out|^2 (LAST = true) into part_out.
// With several workgroups per tile (blockIdx.y: groups of basis vectors for
// the dots) each updates the tile for itself and the first one stores it; in
// and out differ then.  h goes to hout, which may be hsum (the same values),
// and part_out may be part_in when it is not read (no folding).
template <typename W, bool LAST>
__global__ __launch_bounds__(kGT) void k_gs_update(const double* __restrict__ Q, int64_t ldq,
                                                   const int64_t* __restrict__ jd, int nk,
                                                   const W* in, double* out, GsShape G,
                                                   const double* part_in, const double* hsum,
                                                   double* hout, double* part_out) {
  __shared__ double ws[kGsElems];
  __shared__ double hl[kGsH];
  __shared__ double half[kGT];
  const int nv = jd ? (int)jd[0] + 1 : nk;
  const int nr = G.nr;
  const int k0 = LAST ? 0 : (gridDim.y > 1 ? blockIdx.y * kGsVecs : 0);
  const int k1 = LAST ? 0 : (gridDim.y > 1 ? min(k0 + kGsVecs, nv) : nv);
  if (!LAST && k0 >= nv) return;                        // uniform over the workgroup
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t r0 = (int64_t)blockIdx.x * G.tr, r1 = min(r0 + G.tr, G.n);
  const int sr = kGsElems / nr;
  const int kc = kGsH / nr;                             // vectors whose h fits (nr <= 256)
  for (int64_t r = r0; r < r1; r += sr) {
    const int cnt = (int)min((int64_t)sr, r1 - r) * nr;
    const int64_t e0 = r * nr;
    // pieces of at most 128 elements: two threads per element, each half of
    // the vectors of a chunk
    const bool two = cnt <= kGT / 2;
    __syncthreads();                                    // the previous piece is consumed
    for (int e = threadIdx.x; e < cnt; e += kGT) ws[e] = (double)in[e0 + e];
    double acc = 0.0;
    for (int kb = 0; kb < nv; kb += kc) {
      const int ke = min(kb + kc, nv);
      __syncthreads();                                  // the previous chunk is consumed
      if (G.fold) {
        for (int i = wave; i < (ke - kb) * nr; i += kGT / 64) {
          const double v = gs_tile_sum(part_in, (int64_t)kb * nr + i, G.tiles);
          if (lane == 0) hl[i] = v;
        }
      } else {
        for (int i = threadIdx.x; i < (ke - kb) * nr; i += kGT) hl[i] = hsum[(int64_t)kb * nr + i];
      }
      __syncthreads();
      if (blockIdx.x == 0 && blockIdx.y == 0 && r == r0)
        for (int i = threadIdx.x; i < (ke - kb) * nr; i += kGT) hout[(int64_t)kb * nr + i] = hl[i];
      if (two) {
        const int e = threadIdx.x & (kGT / 2 - 1), g = threadIdx.x / (kGT / 2);
        if (e < cnt) {
          const int c = e % nr;
#pragma unroll 8
          for (int k = kb + g; k < ke; k += 2) acc += Q[(int64_t)k * ldq + e0 + e] * hl[(k - kb) * nr + c];
        }
      } else {
        for (int e = threadIdx.x; e < cnt; e += kGT) {
          const int c = e % nr;
          double v = ws[e];
#pragma unroll 8
          for (int k = kb; k < ke; ++k) v -= Q[(int64_t)k * ldq + e0 + e] * hl[(k - kb) * nr + c];
          ws[e] = v;
        }
      }
    }
    if (two) {
      half[threadIdx.x] = acc;
      __syncthreads();
      if ((int)threadIdx.x < cnt) ws[threadIdx.x] -= half[threadIdx.x] + half[threadIdx.x + kGT / 2];
    }
    __syncthreads();
    if (blockIdx.y == 0)
      for (int e = threadIdx.x; e < cnt; e += kGT) out[e0 + e] = ws[e];
    if (!LAST) {
      gs_dots(Q, ldq, k0, k1, ws, e0, cnt, nr, G.tiles, blockIdx.x, r > r0, part_out);
    } else {
      for (int c = wave; c < nr; c += kGT / 64) {
        double v = 0.0;
        for (int e = lane * nr + c; e < cnt; e += 64 * nr) v += ws[e] * ws[e];
        v = wsum(v);
        if (lane == 0) {
          double* o = part_out + (int64_t)c * G.tiles + blockIdx.x;
          *o = r > r0 ? *o + v : v;
        }
      }
    }
  }
}

// The dots and the updates of coarse tiles: partial dots of one vector and one
// tile per workgroup (thread = column and row group), and out = in - Q h over
// all elements.
template <typename W>
__global__ __launch_bounds__(kGT) void k_gs_dots(const double* __restrict__ Q, int64_t ldq,
                                                 const int64_t* __restrict__ jd, int nk,
                                                 const W* __restrict__ w, GsShape G,
                                                 double* __restrict__ part) {
  __shared__ double sum[kGT];
  const int k = blockIdx.y;
  if (k >= (jd ? (int)jd[0] + 1 : nk)) return;          // uniform over the workgroup
  const double* q = Q + (int64_t)k * ldq;
  const int per = kGT / G.nr, c = threadIdx.x % G.nr, r0 = threadIdx.x / G.nr;   // nr <= 256
  double acc = 0.0;
  if (r0 < per) {
    const int64_t end = min((int64_t)(blockIdx.x + 1) * G.tr, G.n);
#pragma unroll 4
    for (int64_t i = (int64_t)blockIdx.x * G.tr + r0; i < end; i += per)
      acc += q[i * G.nr + c] * (double)w[i * G.nr + c];
  }
  sum[threadIdx.x] = acc;
  for (int s = 1; s < per; s <<= 1) {
    __syncthreads();
    if (r0 % (2 * s) == 0 && r0 + s < per) sum[threadIdx.x] += sum[threadIdx.x + s * G.nr];
  }
  if (r0 == 0) part[((int64_t)k * G.nr + c) * G.tiles + blockIdx.x] = sum[threadIdx.x];
}
template <typename W>
__global__ __launch_bounds__(kGT) void k_gs_sub(const double* __restrict__ Q, int64_t ldq,
                                                const int64_t* __restrict__ jd, int nk, const W* in,
                                                const double* __restrict__ h, int nr, double* out) {
  const int nv = jd ? (int)jd[0] + 1 : nk;
  for (int64_t e = blockIdx.x * (int64_t)kGT + threadIdx.x; e < ldq;
       e += (int64_t)gridDim.x * kGT) {
    const int c = (int)(e % nr);
    double v = (double)in[e];
#pragma unroll 4
    for (int k = 0; k < nv; ++k) v -= Q[(int64_t)k * ldq + e] * h[(int64_t)k * nr + c];
    out[e] = v;
  }
}

// out[e] = sum of the tiles of part[e * tiles + t], one wavefront per output.
__global__ __launch_bounds__(256) void k_gs_final(const double* __restrict__ part,
                                                  const int64_t* __restrict__ jd, int nk, int nr,
                                                  int tiles, double* __restrict__ out) {
  const int nv = jd ? (int)jd[0] + 1 : nk;
  const int e = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (e >= nv * nr) return;                             // uniform over the wavefront
  const double s = gs_tile_sum(part, e, tiles);
  if ((threadIdx.x & 63) == 0) out[e] = s;
}

// q = w / |w| into basis vector j + 1 and into the next product's input (xq,
// double or float; may be null), 0 for a column whose norm is 0 or not finite
// (the host ends such a column).  |w|^2 is the sum of part (fold) or nsum.  The
// first workgroup also writes the step's coefficients h1 + h2 and |w| per column
// to res ([(j + 1) nr], [nr]) and
// then, if seq is given, the number seqv + j + 1 to *seq: res and seq are
// then host memory that the host polls (else res is device memory whose
// coefficients may be h1 itself).
template <typename X>
__global__ __launch_bounds__(kGT) void k_gs_next(double* __restrict__ Q, int64_t ldq,
                                                 const int64_t* __restrict__ jd, int j0,
                                                 const double* __restrict__ w, GsShape G,
                                                 const double* __restrict__ part,
                                                 const double* __restrict__ nsum, const double* h1,
                                                 const double* h2, X* __restrict__ xq, double* res,
                                                 int64_t res_slot, int64_t* seq, int64_t seqv) {
  __shared__ double hn[256];                            // nr <= 256
  const int j = jd ? (int)jd[0] : j0;
  if (jd) seqv = jd[1];
  const int nr = G.nr, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int c = wave; c < nr; c += kGT / 64) {
    const double v = G.fold ? gs_tile_sum(part, c, G.tiles) : nsum[c];
    if (lane == 0) hn[c] = v < 0.0 ? 0.0 : sqrt(v);     // NaN stays NaN
  }
  __syncthreads();
  if (blockIdx.x == 0) {
    double* o = res + (int64_t)(j & 1) * res_slot;
    for (int i = threadIdx.x; i < (j + 1) * nr; i += kGT) o[nr + i] = h1[i] + h2[i];
    for (int i = threadIdx.x; i < nr; i += kGT) o[i] = hn[i];
    if (seq) {
      __threadfence_system();
      __syncthreads();
      if (threadIdx.x == 0)
        __hip_atomic_store(seq, seqv + j + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
  }
  double* q = Q + (int64_t)(j + 1) * ldq;
  for (int64_t e = blockIdx.x * (int64_t)kGT + threadIdx.x; e < ldq;
       e += (int64_t)gridDim.x * kGT) {
    const double h = hn[e % nr];
    const double v = h > 0.0 && h < HUGE_VAL ? w[e] * (1.0 / h) : 0.0;
    q[e] = v;
    if (xq) xq[e] = (X)v;
  }
}

// q0 = r * scale per column, into the basis and the product's input; 0 where
// the scale is (also if r is not finite).
template <typename X>
__global__ __launch_bounds__(kGT) void k_gs_start(const double* __restrict__ r,
                                                  const double* __restrict__ sc, int64_t tot,
                                                  int nr, double* __restrict__ q,
                                                  X* __restrict__ xq, int64_t* jd, int64_t seqv) {
  for (int64_t e = blockIdx.x * (int64_t)kGT + threadIdx.x; e < tot;
       e += (int64_t)gridDim.x * kGT) {
    const double f = sc[e % nr];
    const double v = f != 0.0 ? r[e] * f : 0.0;
    q[e] = v;
    if (xq) xq[e] = (X)v;
  }
  if (jd && blockIdx.x == 0 && threadIdx.x == 0) {      // graph replays count their steps here
    jd[0] = 0;
    jd[1] = seqv;
  }
}
__global__ void k_gs_advance(int64_t* jd) {
  if (threadIdx.x == 0) jd[0] += 1;
}

// x[i][c] += sum_{k < nk} Q[k][i][c] y[k][c]
__global__ void k_combine(const double* __restrict__ Q, int64_t ldq, const double* __restrict__ y,
                          int nk, int64_t n, int nr, double* __restrict__ x) {
  const int64_t tot = n * nr;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < tot;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int c = (int)(e % nr);
    double v = x[e];
    for (int k = 0; k < nk; ++k) v += Q[(int64_t)k * ldq + e] * y[k * nr + c];
    x[e] = v;
  }
}

// out[i][c] = a[i][c] * s[c]
__global__ void k_scale_cols(const double* __restrict__ a, const double* __restrict__ s, int64_t n,
                             int nr, double* __restrict__ out) {
  const int64_t tot = n * nr;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < tot;
       e += (int64_t)gridDim.x * blockDim.x)
    out[e] = a[e] * s[e % nr];
}

// out = a + b
__global__ void k_add(const double* __restrict__ a, const double* __restrict__ b, int64_t tot,
                      double* __restrict__ out) {
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < tot;
       e += (int64_t)gridDim.x * blockDim.x)
    out[e] = a[e] + b[e];
}

// out = a - b
__global__ void k_sub(const double* __restrict__ a, const double* __restrict__ b, int64_t tot,
                      double* __restrict__ out) {
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < tot;
       e += (int64_t)gridDim.x * blockDim.x)
    out[e] = a[e] - b[e];
}

template <typename S, typename D>
__global__ void k_convert(const S* __restrict__ a, int64_t tot, D* __restrict__ out) {
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < tot;
       e += (int64_t)gridDim.x * blockDim.x)
    out[e] = (D)a[e];
}

// ---- conjugate gradients (Sec. 4.1), every column its own recurrence.
// alpha_c = rr[c] / pq[c] for active columns (0 for inactive ones and for
// pq = 0); x += alpha p, r -= alpha q.
__global__ void k_cg_update(double* __restrict__ x, double* __restrict__ r,
                            const double* __restrict__ p, const double* __restrict__ q,
                            const double* __restrict__ rr, const double* __restrict__ pq,
                            const double* __restrict__ active, int64_t n, int nr) {
  const int64_t tot = n * nr;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < tot;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int c = (int)(e % nr);
    const double a = (active[c] != 0.0 && pq[c] != 0.0) ? rr[c] / pq[c] : 0.0;
    x[e] += a * p[e];
    r[e] -= a * q[e];
  }
}

// p = r + beta p with beta_c = rr_new[c] / rr_old[c], active columns only.
__global__ void k_cg_dir(double* __restrict__ p, const double* __restrict__ r,
                         const double* __restrict__ rr_new, const double* __restrict__ rr_old,
                         const double* __restrict__ active, int64_t n, int nr) {
  const int64_t tot = n * nr;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < tot;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int c = (int)(e % nr);
    if (active[c] != 0.0 && rr_old[c] != 0.0) p[e] = r[e] + (rr_new[c] / rr_old[c]) * p[e];
  }
}

// ------------------------------------------------------------------ launchers
void cg_update(double* x, double* r, const double* p, const double* q, const double* rr,
               const double* pq, const double* active, int64_t n, int nr, hipStream_t s) {
  k_cg_update<<<grid_for(n * nr, 256, 8192), 256, 0, s>>>(x, r, p, q, rr, pq, active, n, nr);
  HM_LAUNCH_CHECK();
}
void cg_dir(double* p, const double* r, const double* rr_new, const double* rr_old,
            const double* active, int64_t n, int nr, hipStream_t s) {
  k_cg_dir<<<grid_for(n * nr, 256, 8192), 256, 0, s>>>(p, r, rr_new, rr_old, active, n, nr);
  HM_LAUNCH_CHECK();
}
// The orthogonalisation of step j (or jd[0] in a capture) after the product
// win = op(H) q_j, and the next basis vector.  nkmax: basis vectors the
// grids cover (j + 1, or the most a replay can need).
template <typename W, typename X>
static void gs_arnoldi(const GsArgs& a, const W* win, X* xq, int j, int nkmax, hipStream_t s) {
  const GsShape& G = a.G;
  const int64_t tot = G.n * G.nr;
  const int nk = j + 1;
  const unsigned kg = (unsigned)ceil_div(nkmax, kGsVecs);
  const unsigned fin = (unsigned)ceil_div((int64_t)nkmax * G.nr, 4);
  double *h1 = a.h1, *h2 = a.h2;
  auto total = [&](const double* part, int cnt, const int64_t* jd, double* out) {
    if (G.fold) return;
    k_gs_final<<<fin, 256, 0, s>>>(part, jd, cnt, G.nr, G.tiles, out);
    HM_LAUNCH_CHECK();
  };
  if (G.coarse) {
    // 16 columns at N = 9,978 are five tiles, which below would be a workgroup
    // each (restart 100, 44 steps: 48 ms below, 8.3 here, 8.6 with fine tiles; 64
    // columns at N = 1,280, one tile, restart 196, 31 steps: 79 and 8.8)
    const dim3 g(G.tiles, nkmax);
    const unsigned ge = grid_for(tot, kGT, 8192);
    k_gs_dots<W><<<g, kGT, 0, s>>>(a.Q, tot, a.jd, nk, win, G, a.part);
    HM_LAUNCH_CHECK();
    total(a.part, nk, a.jd, h1);
    k_gs_sub<W><<<ge, kGT, 0, s>>>(a.Q, tot, a.jd, nk, win, h1, G.nr, a.w1);
    HM_LAUNCH_CHECK();
    k_gs_dots<double><<<g, kGT, 0, s>>>(a.Q, tot, a.jd, nk, a.w1, G, a.part);
    HM_LAUNCH_CHECK();
    total(a.part, nk, a.jd, h2);
    k_gs_sub<double><<<ge, kGT, 0, s>>>(a.Q, tot, a.jd, nk, a.w1, h2, G.nr, a.w1);
    HM_LAUNCH_CHECK();
    k_gs_dots<double><<<dim3(G.tiles, 1), kGT, 0, s>>>(a.w1, tot, nullptr, 1, a.w1, G, a.part);
    HM_LAUNCH_CHECK();
  } else {
    k_gs_first<W><<<dim3(G.tiles, kg), kGT, 0, s>>>(a.Q, tot, a.jd, nk, win, G, a.part);
    HM_LAUNCH_CHECK();
    total(a.part, nk, a.jd, h2);
    // several workgroups per tile only where tiles alone leave the chip idle:
    // each repeats the update, which reads the whole basis
    k_gs_update<W, false><<<dim3(G.tiles, G.fold ? kg : 1), kGT, 0, s>>>(
        a.Q, tot, a.jd, nk, win, a.w1, G, a.part, h2, h1, a.part2);
    HM_LAUNCH_CHECK();
    total(a.part2, nk, a.jd, h2);
    k_gs_update<double, true><<<dim3(G.tiles, 1), kGT, 0, s>>>(a.Q, tot, a.jd, nk, a.w1, a.w1, G,
                                                               a.part2, h2, h2, a.part);
    HM_LAUNCH_CHECK();
  }
  total(a.part, 1, nullptr, a.nsum);
  k_gs_next<X><<<grid_for(tot, kGT, 2048), kGT, 0, s>>>(a.Q, tot, a.jd, j, a.w1, G, a.part,
                                                        a.nsum, h1, h2, xq, a.res, a.res_slot, a.seq,
                                                        a.seqv);
  HM_LAUNCH_CHECK();
  if (a.jd) {
    k_gs_advance<<<1, 64, 0, s>>>(a.jd);
    HM_LAUNCH_CHECK();
  }
}
void gmres_arnoldi(const GsArgs& a, int j, int nkmax, hipStream_t s) {
  if (a.wf)
    gs_arnoldi<float, float>(a, a.wf, a.xf, j, nkmax, s);
  else
    gs_arnoldi<double, double>(a, a.w, a.xin, j, nkmax, s);
}
void gmres_start(const GsArgs& a, const double* r, const double* sc, hipStream_t s) {
  const int64_t tot = a.G.n * a.G.nr;
  const unsigned g = grid_for(tot, kGT, 2048);
  if (a.wf)
    k_gs_start<float><<<g, kGT, 0, s>>>(r, sc, tot, a.G.nr, a.Q, a.xf, a.jd, a.seqv);
  else
    k_gs_start<double><<<g, kGT, 0, s>>>(r, sc, tot, a.G.nr, a.Q, a.xin, a.jd, a.seqv);
  HM_LAUNCH_CHECK();
}
// out[k nr + c] = Q_k . w per column
void gmres_dots(const double* Q, int nk, const double* w, const GsShape& G, double* part,
                double* out, hipStream_t s) {
  k_gs_first<double><<<dim3(G.tiles, (unsigned)ceil_div(nk, kGsVecs)), kGT, 0, s>>>(
      Q, G.n * G.nr, nullptr, nk, w, G, part);
  HM_LAUNCH_CHECK();
  k_gs_final<<<(unsigned)ceil_div((int64_t)nk * G.nr, 4), 256, 0, s>>>(part, nullptr, nk, G.nr,
                                                                       G.tiles, out);
  HM_LAUNCH_CHECK();
}
void gmres_combine(const double* Q, int64_t ldq, const double* y, int nk, int64_t n, int nr,
                   double* x, hipStream_t s) {
  k_combine<<<grid_for(n * nr, 256, 8192), 256, 0, s>>>(Q, ldq, y, nk, n, nr, x);
  HM_LAUNCH_CHECK();
}
void gmres_scale_cols(const double* a, const double* sc, int64_t n, int nr, double* out,
                      hipStream_t s) {
  k_scale_cols<<<grid_for(n * nr, 256, 8192), 256, 0, s>>>(a, sc, n, nr, out);
  HM_LAUNCH_CHECK();
}
void gmres_sub(const double* a, const double* b, int64_t tot, double* out, hipStream_t s) {
  k_sub<<<grid_for(tot, 256, 8192), 256, 0, s>>>(a, b, tot, out);
  HM_LAUNCH_CHECK();
}
void gmres_add(const double* a, const double* b, int64_t tot, double* out, hipStream_t s) {
  k_add<<<grid_for(tot, 256, 8192), 256, 0, s>>>(a, b, tot, out);
  HM_LAUNCH_CHECK();
}
void convert_f32_to_f64(const float* a, int64_t tot, double* out, hipStream_t s) {
  k_convert<float, double><<<grid_for(tot, 256, 8192), 256, 0, s>>>(a, tot, out);
  HM_LAUNCH_CHECK();
}
void convert_f64_to_f32(const double* a, int64_t tot, float* out, hipStream_t s) {
  k_convert<double, float><<<grid_for(tot, 256, 8192), 256, 0, s>>>(a, tot, out);
  HM_LAUNCH_CHECK();
}

}  // namespace hm
