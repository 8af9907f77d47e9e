// Kernels of the kernel-ridge-regression consumer (Sec. 4.2), binary64:
// k-means, the exact dense kernel matvec (off-diagonal blocks, predictions),
// the block-diagonal preconditioner (dense blocks, Cholesky, inverse, batched
// GEMV) and the conjugate-gradient vector and scalar updates.  Every
// reduction runs in a fixed order, so results do not depend on scheduling.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "krr_kernels.hpp"

namespace hdf {
namespace krr {

namespace {

constexpr int kMaxK = 256;

template <int KIND>
__device__ __forceinline__ double kval(double r2, double a) {
  // a: 1/(2 l^2) Gaussian, 1/l^2 Cauchy, sqrt(3)/l Matern-3/2, sqrt(5)/l Matern-5/2
  if constexpr (KIND == 0) {
    return exp(-r2 * a);
  } else if constexpr (KIND == 1) {
    return 1.0 / (1.0 + r2 * a);
  } else if constexpr (KIND == 2) {
    const double z = sqrt(r2) * a;
    return (1.0 + z) * exp(-z);
  } else {
    const double z = sqrt(r2) * a;
    return (1.0 + z + z * z / 3.0) * exp(-z);
  }
}

double kernel_param(int kind, double l) {
  switch (kind) {
    case 0: return 1.0 / (2.0 * l * l);
    case 1: return 1.0 / (l * l);
    case 2: return 1.7320508075688772 / l;
    default: return 2.23606797749979 / l;
  }
}

// Sum of part[0..np) in a fixed order over one 256-thread block; every
// thread gets the result.
__device__ double block_sum(const double* part, int np, double* sh) {
  double s = 0.0;
  for (int t = threadIdx.x; t < np; t += 256) s += part[t];
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
    __syncthreads();
  }
  const double r = sh[0];
  __syncthreads();
  return r;
}

// Tree sum of one value per thread of a 256-thread block, written by thread 0.
__device__ void block_store(double v, double* sh, double* out) {
  sh[threadIdx.x] = v;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = sh[0];
}

// ---------------------------------------------------------------- k-means

__global__ __launch_bounds__(256) void k_gather_rows(const double* __restrict__ x, int64_t ld,
                                                     const int64_t* __restrict__ idx, int64_t m, int d,
                                                     double* __restrict__ out, int64_t ldo) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= m * d) return;
  const int64_t i = e / d;
  const int t = (int)(e % d);
  out[i * ldo + t] = x[idx[i] * ld + t];
}

template <int D>
__global__ __launch_bounds__(256) void k_km_assign(const double* __restrict__ x, int64_t ld, int64_t n,
                                                   const double* __restrict__ centres, int k,
                                                   int32_t* __restrict__ labels, int32_t* __restrict__ changed,
                                                   int first) {
#pragma clang fp contract(off)
  __shared__ double sc[kMaxK * D];
  for (int t = threadIdx.x; t < k * D; t += 256) sc[t] = centres[t];
  __syncthreads();
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  int moved = 0;
  if (i < n) {
    double xi[D];
#pragma unroll
    for (int t = 0; t < D; ++t) xi[t] = x[i * ld + t];
    int best = 0;
    double bd = 0.0;
    for (int c = 0; c < k; ++c) {
      double s = 0.0;
#pragma unroll
      for (int t = 0; t < D; ++t) {
        const double u = xi[t] - sc[c * D + t];
        const double u2 = u * u;
        s = s + u2;
      }
      if (c == 0 || s < bd) {
        bd = s;
        best = c;
      }
    }
    moved = first ? 1 : (labels[i] != best);
    labels[i] = best;
  }
  const int cnt = __syncthreads_count(moved);
  if (threadIdx.x == 0) changed[blockIdx.x] = cnt;
}

constexpr int kKmChunk = 4096;

// part[(c * chunks + b) * (D + 1) + t]: sum of coordinate t (t = D: count) of
// the members of c among points [b * kKmChunk, (b + 1) * kKmChunk)
template <int D>
__global__ __launch_bounds__(256) void k_km_partial(const double* __restrict__ x, int64_t ld, int64_t n,
                                                    const int32_t* __restrict__ labels, double* __restrict__ part) {
  __shared__ double sh[256];
  const int c = blockIdx.x;
  const int b = blockIdx.y;
  const int64_t i0 = (int64_t)b * kKmChunk;
  const int64_t i1 = min(n, i0 + kKmChunk);
  double acc[D + 1];
#pragma unroll
  for (int t = 0; t <= D; ++t) acc[t] = 0.0;
  for (int64_t i = i0 + threadIdx.x; i < i1; i += 256) {
    if (labels[i] == c) {
#pragma unroll
      for (int t = 0; t < D; ++t) acc[t] += x[i * ld + t];
      acc[D] += 1.0;
    }
  }
  double* out = part + ((int64_t)c * gridDim.y + b) * (D + 1);
#pragma unroll
  for (int t = 0; t <= D; ++t) {
    block_store(acc[t], sh, out + t);
    __syncthreads();
  }
}

template <int D>
__global__ __launch_bounds__(256) void k_km_finish(const double* __restrict__ part, int chunks, int k,
                                                   double* __restrict__ centres) {
  const int c = threadIdx.x;
  if (c >= k) return;
  double acc[D + 1];
#pragma unroll
  for (int t = 0; t <= D; ++t) acc[t] = 0.0;
  for (int b = 0; b < chunks; ++b) {
    const double* p = part + ((int64_t)c * chunks + b) * (D + 1);
#pragma unroll
    for (int t = 0; t <= D; ++t) acc[t] += p[t];
  }
  if (acc[D] > 0.0) {
#pragma unroll
    for (int t = 0; t < D; ++t) centres[c * D + t] = acc[t] / acc[D];
  }
}

// ------------------------------------------------------ dense kernel matvec

template <int D, int KIND, bool MASK>
__global__ __launch_bounds__(256) void k_kmv(const double* __restrict__ x, int64_t ldx, int nx,
                                             const double* __restrict__ y, int64_t ldy, int ny,
                                             const double* __restrict__ w, const int32_t* __restrict__ lohi,
                                             double ka, int chunk, double* __restrict__ part) {
  __shared__ double sy[D][256];
  __shared__ double sw[256];
  const int i = blockIdx.x * 256 + threadIdx.x;
  const int j0 = (int)min((int64_t)ny, (int64_t)blockIdx.y * chunk);
  const int j1 = (int)min((int64_t)ny, (int64_t)j0 + chunk);
  double xi[D];
  int lo = 0, hi = 0;
  if (i < nx) {
#pragma unroll
    for (int t = 0; t < D; ++t) xi[t] = x[(int64_t)i * ldx + t];
    if (MASK) {
      lo = lohi[2 * i];
      hi = lohi[2 * i + 1];
    }
  } else {
#pragma unroll
    for (int t = 0; t < D; ++t) xi[t] = 0.0;
  }
  double acc = 0.0;
  for (int jb = j0; jb < j1; jb += 256) {
    const int j = jb + threadIdx.x;
    __syncthreads();
    if (j < j1) {
#pragma unroll
      for (int t = 0; t < D; ++t) sy[t][threadIdx.x] = y[(int64_t)j * ldy + t];
      sw[threadIdx.x] = w[j];
    }
    __syncthreads();
    const int cnt = min(256, j1 - jb);
#pragma unroll 4
    for (int jj = 0; jj < cnt; ++jj) {
      double r2 = 0.0;
#pragma unroll
      for (int t = 0; t < D; ++t) {
        const double u = xi[t] - sy[t][jj];
        r2 = fma(u, u, r2);
      }
      const double kv = kval<KIND>(r2, ka);
      double c = sw[jj];
      if (MASK) c = (jb + jj >= lo && jb + jj < hi) ? 0.0 : c;
      acc = fma(kv, c, acc);
    }
  }
  if (i < nx) part[(int64_t)blockIdx.y * nx + i] = acc;
}

// 64 entries per workgroup, wavefront w takes the partial sums w, w + 4, ... (a fixed order)
__global__ __launch_bounds__(256) void k_kmv_finish(const double* __restrict__ part, int splits, int64_t n,
                                                    const double* __restrict__ base, const double* __restrict__ v,
                                                    double lam, double* __restrict__ out,
                                                    double* __restrict__ part_dot) {
  __shared__ double red[4][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t i = (int64_t)blockIdx.x * 64 + lane;
  double acc[4] = {0, 0, 0, 0};
  if (i < n) {
    int k = w;
    for (; k + 12 < splits; k += 16)
#pragma unroll
      for (int u = 0; u < 4; ++u) acc[u] += part[(int64_t)(k + 4 * u) * n + i];
    for (; k < splits; k += 4) acc[0] += part[(int64_t)k * n + i];
  }
  red[w][lane] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
  __syncthreads();
  if (w != 0) return;
  double dot = 0.0;
  if (i < n) {
    double s = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
    if (base) s += base[i];
    if (v) {
      s = fma(lam, v[i], s);
      dot = v[i] * s;
    }
    out[i] = s;
  }
  if (part_dot) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) dot += __shfl_xor(dot, off);
    if (lane == 0) part_dot[blockIdx.x] = dot;
  }
}

__global__ __launch_bounds__(256) void k_gather(const double* __restrict__ v, const int32_t* __restrict__ perm,
                                                int64_t n, double* __restrict__ out) {
  const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (p < n) out[p] = v[perm[p]];
}

__global__ __launch_bounds__(256) void k_scatter(const double* __restrict__ v, const int32_t* __restrict__ perm,
                                                 int64_t n, double* __restrict__ out) {
  const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (p < n) out[perm[p]] = v[p];
}

// ---------------------------------------------------- preconditioner blocks

// Upper tiles (tile row <= tile column) of lam I + K for each block, in rows of 64 nt; the rows and
// columns past the block's n are those of the identity.
template <int D, int KIND>
__global__ __launch_bounds__(256) void k_dense_blocks(const double* __restrict__ xs, const Block* __restrict__ blocks,
                                                      double ka, double lam, double* __restrict__ M) {
  const Block B = blocks[blockIdx.y];
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int np = kTile * B.nt;
  if (e >= (int64_t)np * np) return;
  const int i = (int)(e / np), j = (int)(e % np);
  if (i / kTile > j / kTile) return;
  double v = i == j ? 1.0 : 0.0;
  if (i < B.n && j < B.n) {
    const double* xi = xs + (B.pos + i) * D;
    const double* xj = xs + (B.pos + j) * D;
    double r2 = 0.0;
#pragma unroll
    for (int t = 0; t < D; ++t) {
      const double u = xi[t] - xj[t];
      r2 = fma(u, u, r2);
    }
    v = kval<KIND>(r2, ka) + (i == j ? lam : 0.0);
  }
  M[B.poff + e] = v;
}

// Inverses of the preconditioner's blocks: A = U^T U by elimination on [A | I], tile by tile, then
// A^-1 = L^-T L^-1 with L = U^T.  Work storage of a block (64 nt square): its upper tiles hold A and
// then the rows of U, its strictly lower tiles L^-1 as the elimination forms it, its diagonal tiles
// the inverses of the diagonal factors, (L_jj)^-1.  Step j of the elimination, over all blocks at once:
//   k_inv_panel  M_jt <- (L_jj)^-1 M_jt          for every tile t != j of row j, by substitution
//   k_inv_trail  M_ci -= M_jc^T M_ji             for c > j and i <= j (L^-1) or i >= c (A), and the
//                                                workgroup of M_(j+1)(j+1) factorises that tile next
// so a block of n points costs 2 nt launches of up to nt^2 / 4 workgroups, the bulk of the work (the
// trail and the final product) on the matrix cores, and the serial 64-step factorisation of a
// diagonal tile overlaps the other tiles' updates.  What bounds it is that chain of steps.  The
// preconditioner of 13,760 points in 30 blocks of up to 777 (allocations included): 146.6 ms with one
// workgroup per block and one thread per column of the inverse, 2.07 ms so.
// Every entry takes its products one by one in the order of the steps, each subtracted with one
// rounding: the entries of a kernel matrix shrink as the elimination goes on, and a sum of 64 products
// formed first, or a panel formed with the explicit inverse of the diagonal factor, is rounded at its
// own, larger size (z = A^-1 r of 13,760 points in 30 blocks, against extended precision: 4.7e-14 so,
// 6.4e-15 in this order).
typedef double doublex2 __attribute__((ext_vector_type(2)));
typedef double doublex4 __attribute__((ext_vector_type(4)));
constexpr int kTS = 80;                               // LDS row stride: rows k and k + 1 on different bank halves
constexpr int kTileLds = kTile * kTS;                 // doubles of a staged tile

// a 64 x 64 tile with row stride ld into LDS (256 threads, 16-byte loads)
__device__ __forceinline__ void tile_load(const double* __restrict__ src, int64_t ld, double* __restrict__ dst) {
#pragma unroll
  for (int it = 0; it < 8; ++it) {
    const int e = it * 256 + threadIdx.x;
    const int row = e >> 5, c2 = (e & 31) * 2;
    *reinterpret_cast<doublex2*>(dst + row * kTS + c2) = *reinterpret_cast<const doublex2*>(src + row * ld + c2);
  }
}

// acc += SIGN P^T Q: wavefront w forms rows 16 w .. 16 w + 15, four 16 x 16 accumulator tiles
template <int SIGN>
__device__ __forceinline__ void tile_product(const double* P, const double* Q, doublex4 (&acc)[4]) {
  const int lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4, w = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < kTile; k += 4) {
    const double a = SIGN * P[(k + q) * kTS + 16 * w + r];
#pragma unroll
    for (int t = 0; t < 4; ++t)
      acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, Q[(k + q) * kTS + 16 * t + r], acc[t], 0, 0, 0);
  }
}

constexpr int kDiag = kTile * kTile + kTile;          // a diagonal factor U_jj and its reciprocal diagonal

// Factorisation of the diagonal tile in registers: thread (w, l) holds rows 16 w .. 16 w + 15 of
// column l of the tile and of the identity.  The wavefront that owns row j scales it and publishes
// the rows of U and L^-1 in `rows` (LDS, 2 x 192 values); one barrier per step.
__device__ void tile_factor(double (&a)[16], double* rows, int j0, int32_t* status, double* Mjj, int64_t ld,
                            double* dj) {
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  double b[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) b[q] = 16 * w + q == l ? 1.0 : 0.0;
  int bad = 0;
  // row j (row q of this wavefront): pivot from lane j by way of LDS, both parts divided by its root
  auto publish = [&](int j, double& aq, double& bq) {
    double* next = rows + 192 * (j & 1);
    next[128 + l] = aq;
    __builtin_amdgcn_wave_barrier();
    double p = next[128 + j];
    if (!(p > 0.0 && p < INFINITY)) {
      if (!bad) bad = j0 + j + 1;
      p = 1.0;
    }
    const double d = sqrt(p);
    aq /= d;
    bq /= d;
    next[l] = aq;
    next[64 + l] = bq;
    if (l == j) dj[kTile * kTile + j] = 1.0 / d;
  };
  if (w == 0) publish(0, a[0], b[0]);
  __syncthreads();
  for (int wj = 0; wj < 4; ++wj) {
#pragma unroll
    for (int jj = 0; jj < 16; ++jj) {
      const int j = 16 * wj + jj;
      const double* row = rows + 192 * (j & 1);
      if (w >= wj) {
        const double ra = row[l], rb = row[64 + l];
#pragma unroll
        for (int q = 0; q < 16; ++q) {
          if (w > wj || q > jj) {
            const double m = -row[16 * w + q];
            a[q] = fma(m, ra, a[q]);
            b[q] = fma(m, rb, b[q]);
          }
        }
      }
      if (jj < 15) {
        if (w == wj) publish(j + 1, a[(jj + 1) & 15], b[(jj + 1) & 15]);
      } else if (w == wj + 1) {
        publish(j + 1, a[0], b[0]);
      }
      __syncthreads();
    }
  }
  // the wavefronts own consecutive rows: the first bad step is the lowest of theirs
  int* first = reinterpret_cast<int*>(rows);
  if (l == 0) first[w] = bad;
  __syncthreads();
  if (threadIdx.x == 0 && *status == 0) {
    for (int v = 3; v >= 0; --v) bad = first[v] ? first[v] : bad;
    if (bad) *status = bad;
  }
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int row = 16 * w + q;
    Mjj[row * ld + l] = b[q];
    dj[row * kTile + l] = a[q];
  }
}

__global__ __launch_bounds__(256) void k_inv_first(double* __restrict__ M, double* __restrict__ diag,
                                                   const Block* __restrict__ blocks, int32_t* __restrict__ status) {
  __shared__ double rows[384];
  const Block B = blocks[blockIdx.x];
  const int64_t ld = (int64_t)kTile * B.nt;
  double* m = M + B.poff;
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  double a[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) a[q] = m[(16 * w + q) * ld + l];
  if (threadIdx.x == 0) status[blockIdx.x] = 0;
  tile_factor(a, rows, 0, status + blockIdx.x, m, ld, diag + B.doff * kDiag);
}

// One wavefront per tile, one column per lane: X = (U_jj)^-T M_jt by forward substitution in
// registers, U_jj read as wavefront-uniform values.  The quotients are formed from the reciprocal
// diagonal with one correction.
__global__ __launch_bounds__(64) void k_inv_panel(double* __restrict__ M, const double* __restrict__ diag,
                                                  const Block* __restrict__ blocks, int j) {
  const Block B = blocks[blockIdx.y];
  if (j >= B.nt || (int)blockIdx.x >= B.nt - 1) return;
  const int t = (int)blockIdx.x < j ? blockIdx.x : blockIdx.x + 1;
  const int64_t ld = (int64_t)kTile * B.nt;
  double* c = M + B.poff + (int64_t)j * kTile * ld + (int64_t)t * kTile + threadIdx.x;
  const double* U = diag + (B.doff + j) * kDiag;
  double x[kTile];
#pragma unroll
  for (int r = 0; r < kTile; ++r) x[r] = c[r * ld];
#pragma unroll
  for (int r = 0; r < kTile; ++r) {
    const double inv = U[kTile * kTile + r];
    double v = x[r] * inv;
    v = fma(fma(-v, U[r * kTile + r], x[r]), inv, v);
    c[r * ld] = v;
#pragma unroll
    for (int k = r + 1; k < kTile; ++k) x[k] = fma(-U[r * kTile + k], v, x[k]);
  }
}

__global__ __launch_bounds__(256) void k_inv_trail(double* __restrict__ M, double* __restrict__ diag,
                                                   const Block* __restrict__ blocks, int j,
                                                   int32_t* __restrict__ status) {
  extern __shared__ unsigned char smem_raw[];
  double* P = reinterpret_cast<double*>(smem_raw);
  double* Q = P + kTileLds;
  const Block B = blocks[blockIdx.y];
  // tiles of the trailing rows c > j: first the upper ones (row j + 1 first), then the j + 1 columns of L^-1
  const int nr = B.nt - 1 - j;
  int x = blockIdx.x, c, i;
  if (nr < 1) return;
  const int64_t upper = (int64_t)nr * (nr + 1) / 2;
  if (x < upper) {
    c = 0;
    while (x >= nr - c) x -= nr - c++;
    i = j + 1 + c + x;
    c += j + 1;
  } else {
    x -= (int)upper;
    if (x >= nr * (j + 1)) return;
    c = j + 1 + x / (j + 1);
    i = x % (j + 1);
  }
  const int64_t ld = (int64_t)kTile * B.nt;
  double* m = M + B.poff;
  const double* rowj = m + (int64_t)j * kTile * ld;
  double* out = m + (int64_t)c * kTile * ld + (int64_t)i * kTile;
  tile_load(rowj + (int64_t)c * kTile, ld, P);
  if (c != i) tile_load(rowj + (int64_t)i * kTile, ld, Q);
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4, w = threadIdx.x >> 6;
  doublex4 acc[4];
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[u][e] = i == j ? 0.0 : out[(16 * w + g + 4 * e) * ld + 16 * u + r];
  __syncthreads();
  tile_product<-1>(P, c != i ? Q : P, acc);
  const bool next = c == i && c == j + 1;             // uniform
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int row = 16 * w + g + 4 * e, col = 16 * u + r;
      if (next) Q[row * kTS + col] = acc[u][e];
      else out[row * ld + col] = acc[u][e];
    }
  if (!next) return;
  __syncthreads();
  const int l = lane;
  double a[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) a[q] = Q[(16 * w + q) * kTS + l];
  tile_factor(a, P, kTile * c, status + blockIdx.y, out, ld, diag + (B.doff + c) * kDiag);
}

// X = L^-T L^-1: tile (i, c), i <= c, sums the tiles k >= c of columns i and c of L^-1; the tile is
// written to both halves of the n x n inverse.
__global__ __launch_bounds__(256) void k_inv_form(const double* __restrict__ M, const Block* __restrict__ blocks,
                                                  double* __restrict__ X) {
  extern __shared__ unsigned char smem_raw[];
  double* P = reinterpret_cast<double*>(smem_raw);
  double* Q = P + kTileLds;
  const Block B = blocks[blockIdx.y];
  int x = blockIdx.x, i = 0;
  if (x >= (int64_t)B.nt * (B.nt + 1) / 2) return;
  while (x >= B.nt - i) x -= B.nt - i++;
  const int c = i + x;
  const int64_t ld = (int64_t)kTile * B.nt;
  const double* m = M + B.poff;
  doublex4 acc[4] = {{0, 0, 0, 0}, {0, 0, 0, 0}, {0, 0, 0, 0}, {0, 0, 0, 0}};
  for (int k = c; k < B.nt; ++k) {
    const double* rowk = m + (int64_t)k * kTile * ld;
    __syncthreads();
    tile_load(rowk + (int64_t)i * kTile, ld, P);
    if (c != i) tile_load(rowk + (int64_t)c * kTile, ld, Q);
    __syncthreads();
    tile_product<1>(P, c != i ? Q : P, acc);
  }
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4, w = threadIdx.x >> 6;
  double* out = X + B.aoff;
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int row = kTile * i + 16 * w + g + 4 * e, col = kTile * c + 16 * u + r;
      if (row < B.n && col < B.n) out[(int64_t)row * B.n + col] = acc[u][e];
    }
  if (c == i) return;
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int e = 0; e < 4; ++e) P[(16 * u + r) * kTS + 16 * w + g + 4 * e] = acc[u][e];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int row = kTile * c + 16 * w + q, col = kTile * i + lane;
    if (row < B.n && col < B.n) out[(int64_t)row * B.n + col] = P[(16 * w + q) * kTS + lane];
  }
}

// One wavefront per row position p of the cluster order.
__global__ __launch_bounds__(256) void k_block_gemv(const double* __restrict__ Ainv, const Block* __restrict__ blocks,
                                                    const int32_t* __restrict__ row_block, int64_t n,
                                                    const double* __restrict__ r, double* __restrict__ z,
                                                    double* __restrict__ part_rz, const CGState* __restrict__ st) {
  if (st && st->done) return;
  __shared__ double sh[4];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t p = (int64_t)blockIdx.x * 4 + wave;
  double contrib = 0.0;
  if (p < n) {
    const Block B = blocks[row_block[p]];
    const int64_t i = p - B.pos;
    const double* row = Ainv + B.aoff + i * B.n;
    const double* rc = r + B.pos;
    double s = 0.0;
    for (int j = lane; j < B.n; j += 64) s = fma(row[j], rc[j], s);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
    if (lane == 0) z[p] = s;
    contrib = r[p] * s;
  }
  if (part_rz) {
    if (lane == 0) sh[wave] = contrib;
    __syncthreads();
    if (threadIdx.x == 0) part_rz[blockIdx.x] = (sh[0] + sh[1]) + (sh[2] + sh[3]);
  }
}

// ------------------------------------------------------ conjugate gradients

__global__ __launch_bounds__(256) void k_dot_partial(const double* __restrict__ a, const double* __restrict__ b,
                                                     int64_t n, double* __restrict__ part) {
  __shared__ double sh[256];
  double s = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)kDotBlocks * 256) s = fma(a[i], b[i], s);
  block_store(s, sh, part + blockIdx.x);
}

__global__ __launch_bounds__(256) void k_cg_start(const double* __restrict__ y, int64_t n, double* __restrict__ x,
                                                  double* __restrict__ r) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  x[i] = 0.0;
  r[i] = y[i];
}

__global__ __launch_bounds__(256) void k_cg_init(CGState* __restrict__ st, const double* __restrict__ part_bb,
                                                 const double* __restrict__ part_rz, int nrz, double rtol2, int max_it) {
  __shared__ double sh[256];
  const double bb = block_sum(part_bb, kDotBlocks, sh);
  const double rz = block_sum(part_rz, nrz, sh);
  if (threadIdx.x == 0) {
    st->bb = bb;
    st->rz = rz;
    st->rr = bb;
    st->rtol2 = rtol2;
    st->beta = 0.0;
    st->it = 0;
    st->max_it = max_it;
    st->done = bb == 0.0 ? 1 : (max_it <= 0 ? 2 : 0);
  }
}

// every workgroup sums the partial p . q for itself: a launch less than a scalar kernel before it
__global__ __launch_bounds__(256) void k_cg_xr(double* __restrict__ x, double* __restrict__ r,
                                               const double* __restrict__ p, const double* __restrict__ q, int64_t n,
                                               const CGState* __restrict__ st, const double* __restrict__ part_pq,
                                               int npq, double* __restrict__ part_rr) {
  if (st->done) return;
  __shared__ double sh[256];
  const double a = st->rz / block_sum(part_pq, npq, sh);
  double s = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)kDotBlocks * 256) {
    x[i] = fma(a, p[i], x[i]);
    const double ri = fma(-a, q[i], r[i]);
    r[i] = ri;
    s = fma(ri, ri, s);
  }
  block_store(s, sh, part_rr + blockIdx.x);
}

__global__ __launch_bounds__(256) void k_cg_step(CGState* __restrict__ st, const double* __restrict__ part_rr,
                                                 const double* __restrict__ part_rz, int nrz) {
  if (st->done) return;
  __shared__ double sh[256];
  const double rr = block_sum(part_rr, kDotBlocks, sh);
  const double rz = block_sum(part_rz, nrz, sh);
  if (threadIdx.x == 0) {
    st->rr = rr;
    const int it = st->it + 1;
    st->it = it;
    if (rr <= st->rtol2 * st->bb) st->done = 1;
    else if (it >= st->max_it) st->done = 2;
    if (!st->done) {
      st->beta = rz / st->rz;
      st->rz = rz;
    }
  }
}

__global__ __launch_bounds__(256) void k_cg_p(double* __restrict__ p, const double* __restrict__ z, int64_t n,
                                              const CGState* __restrict__ st) {
  if (st->done) return;
  const double b = st->beta;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
    p[i] = fma(b, p[i], z[i]);
}

unsigned blocks_for(int64_t n) { return (unsigned)std::max<int64_t>(1, (n + 255) / 256); }

}  // namespace

// ---------------------------------------------------------------- launchers

hipError_t launch_gather_rows(const double* x, int64_t ld, const int64_t* idx, int64_t m, int d, double* out,
                              int64_t ldo, hipStream_t s) {
  k_gather_rows<<<blocks_for(m * d), 256, 0, s>>>(x, ld, idx, m, d, out, ldo);
  return hipGetLastError();
}

#define KRR_DISPATCH_D(d, MACRO) \
  switch (d) {                   \
    case 1: MACRO(1); break;     \
    case 2: MACRO(2); break;     \
    case 3: MACRO(3); break;     \
    case 4: MACRO(4); break;     \
    case 5: MACRO(5); break;     \
    case 6: MACRO(6); break;     \
    case 7: MACRO(7); break;     \
    case 8: MACRO(8); break;     \
    default: return hipErrorInvalidValue; \
  }

hipError_t launch_km_assign(const double* x, int64_t ld, int64_t n, int d, const double* centres, int k,
                            int32_t* labels, int32_t* changed_per_block, int* n_blocks, hipStream_t s) {
  // first call on a labels array: n_blocks < 0 on entry (labels not read)
  const int first = *n_blocks < 0 ? 1 : 0;
  const unsigned g = blocks_for(n);
  *n_blocks = (int)g;
#define KM_A(D) k_km_assign<D><<<g, 256, 0, s>>>(x, ld, n, centres, k, labels, changed_per_block, first)
  KRR_DISPATCH_D(d, KM_A)
#undef KM_A
  return hipGetLastError();
}

int km_update_chunks(int64_t n) { return (int)std::max<int64_t>(1, (n + kKmChunk - 1) / kKmChunk); }

hipError_t launch_km_update(const double* x, int64_t ld, int64_t n, int d, const int32_t* labels, int k,
                            double* part, double* centres, hipStream_t s) {
  const int chunks = km_update_chunks(n);
  const dim3 g((unsigned)k, (unsigned)chunks);
#define KM_U(D)                                                      \
  k_km_partial<D><<<g, 256, 0, s>>>(x, ld, n, labels, part);         \
  k_km_finish<D><<<1, 256, 0, s>>>(part, chunks, k, centres)
  KRR_DISPATCH_D(d, KM_U)
#undef KM_U
  return hipGetLastError();
}

int kmv_splits(int64_t nx, int64_t ny) {
  // enough workgroups to fill the chip, at least 512 columns per split
  const int64_t rows = (nx + 255) / 256;
  int64_t s = std::max<int64_t>(1, 2048 / std::max<int64_t>(1, rows));
  s = std::min<int64_t>(s, std::max<int64_t>(1, ny / 512));
  return (int)std::min<int64_t>(s, 1024);
}

hipError_t launch_kmv(const double* x, int64_t ldx, int64_t nx, const double* y, int64_t ldy, int64_t ny, int d,
                      int kernel, double l, const double* w, const int32_t* lohi, double* part, int splits,
                      hipStream_t s) {
  if (kernel < 0 || kernel > 3 || splits < 1) return hipErrorInvalidValue;
  const int64_t per = (ny + splits - 1) / splits;
  const int chunk = (int)std::max<int64_t>(256, (per + 255) / 256 * 256);
  const dim3 g(blocks_for(nx), (unsigned)splits);
  const double ka = kernel_param(kernel, l);
  const int ix = (int)nx, iy = (int)ny;
#define KMV_K(D, K)                                                                                        \
  do {                                                                                                     \
    if (lohi) k_kmv<D, K, true><<<g, 256, 0, s>>>(x, ldx, ix, y, ldy, iy, w, lohi, ka, chunk, part);       \
    else k_kmv<D, K, false><<<g, 256, 0, s>>>(x, ldx, ix, y, ldy, iy, w, lohi, ka, chunk, part);           \
  } while (0)
#define KMV_D(D)                         \
  switch (kernel) {                      \
    case 0: KMV_K(D, 0); break;          \
    case 1: KMV_K(D, 1); break;          \
    case 2: KMV_K(D, 2); break;          \
    default: KMV_K(D, 3); break;         \
  }
  KRR_DISPATCH_D(d, KMV_D)
#undef KMV_D
#undef KMV_K
  return hipGetLastError();
}

int kmv_finish_blocks(int64_t n) { return (int)std::max<int64_t>(1, (n + 63) / 64); }

hipError_t launch_kmv_finish(const double* part, int splits, int64_t n, const double* base, const double* v,
                             double lam, double* out, double* part_dot, hipStream_t s) {
  k_kmv_finish<<<(unsigned)kmv_finish_blocks(n), 256, 0, s>>>(part, splits, n, base, v, lam, out, part_dot);
  return hipGetLastError();
}

hipError_t launch_gather(const double* v, const int32_t* perm, int64_t n, double* out, hipStream_t s) {
  k_gather<<<blocks_for(n), 256, 0, s>>>(v, perm, n, out);
  return hipGetLastError();
}

hipError_t launch_scatter(const double* v, const int32_t* perm, int64_t n, double* out, hipStream_t s) {
  k_scatter<<<blocks_for(n), 256, 0, s>>>(v, perm, n, out);
  return hipGetLastError();
}

hipError_t launch_dense_blocks(const double* xs, int d, const Block* blocks, int nb, int max_nt, int kernel,
                               double l, double lam, double* M, hipStream_t s) {
  if (kernel < 0 || kernel > 3 || nb < 1) return hipErrorInvalidValue;
  const dim3 g(blocks_for((int64_t)max_nt * kTile * max_nt * kTile), (unsigned)nb);
  const double ka = kernel_param(kernel, l);
#define DB_K(D, K) k_dense_blocks<D, K><<<g, 256, 0, s>>>(xs, blocks, ka, lam, M)
#define DB_D(D)                        \
  switch (kernel) {                    \
    case 0: DB_K(D, 0); break;         \
    case 1: DB_K(D, 1); break;         \
    case 2: DB_K(D, 2); break;         \
    default: DB_K(D, 3); break;        \
  }
  KRR_DISPATCH_D(d, DB_D)
#undef DB_D
#undef DB_K
  return hipGetLastError();
}

hipError_t launch_block_inverse(double* M, double* diag, const Block* blocks, int nb, int max_nt, int32_t* status,
                                double* X, hipStream_t s) {
  if (nb < 1 || max_nt < 1) return hipErrorInvalidValue;
  const size_t lds = 2 * (size_t)kTileLds * sizeof(double);
  k_inv_first<<<(unsigned)nb, 256, 0, s>>>(M, diag, blocks, status);
  for (int j = 0; j < max_nt; ++j) {
    const unsigned nr = (unsigned)(max_nt - 1 - j);
    if (max_nt > 1) k_inv_panel<<<dim3((unsigned)max_nt - 1, (unsigned)nb), 64, 0, s>>>(M, diag, blocks, j);
    if (nr > 0)
      k_inv_trail<<<dim3(nr * (nr + 1) / 2 + nr * (unsigned)(j + 1), (unsigned)nb), 256, lds, s>>>(M, diag, blocks, j,
                                                                                                  status);
  }
  k_inv_form<<<dim3((unsigned)max_nt * ((unsigned)max_nt + 1) / 2, (unsigned)nb), 256, lds, s>>>(M, blocks, X);
  return hipGetLastError();
}

int block_gemv_blocks(int64_t n) { return (int)std::max<int64_t>(1, (n + 3) / 4); }

hipError_t launch_block_gemv(const double* Ainv, const Block* blocks, const int32_t* row_block, int64_t n,
                             const double* r, double* z, double* part_rz, const CGState* st, hipStream_t s) {
  k_block_gemv<<<(unsigned)block_gemv_blocks(n), 256, 0, s>>>(Ainv, blocks, row_block, n, r, z, part_rz, st);
  return hipGetLastError();
}

hipError_t launch_dot_partial(const double* a, const double* b, int64_t n, double* part, hipStream_t s) {
  k_dot_partial<<<kDotBlocks, 256, 0, s>>>(a, b, n, part);
  return hipGetLastError();
}

hipError_t launch_cg_start(const double* y, int64_t n, double* x, double* r, hipStream_t s) {
  k_cg_start<<<blocks_for(n), 256, 0, s>>>(y, n, x, r);
  return hipGetLastError();
}

hipError_t launch_cg_init(CGState* st, const double* part_bb, const double* part_rz, int nrz, double rtol2,
                          int max_it, const double* z, double* p, int64_t n, hipStream_t s) {
  k_cg_init<<<1, 256, 0, s>>>(st, part_bb, part_rz, nrz, rtol2, max_it);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return hipMemcpyAsync(p, z, (size_t)n * sizeof(double), hipMemcpyDeviceToDevice, s);
}

hipError_t launch_cg_xr(double* x, double* r, const double* p, const double* q, int64_t n, const CGState* st,
                        const double* part_pq, int npq, double* part_rr, hipStream_t s) {
  k_cg_xr<<<kDotBlocks, 256, 0, s>>>(x, r, p, q, n, st, part_pq, npq, part_rr);
  return hipGetLastError();
}

hipError_t launch_cg_step(CGState* st, const double* part_rr, const double* part_rz, int nrz, hipStream_t s) {
  k_cg_step<<<1, 256, 0, s>>>(st, part_rr, part_rz, nrz);
  return hipGetLastError();
}

hipError_t launch_cg_p(double* p, const double* z, int64_t n, const CGState* st, hipStream_t s) {
  k_cg_p<<<(unsigned)std::min<int64_t>(blocks_for(n), 1024), 256, 0, s>>>(p, z, n, st);
  return hipGetLastError();
}

}  // namespace krr
}  // namespace hdf
