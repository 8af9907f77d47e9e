// gfx950 kernels of the HDF hot path: geometry, radial Gram moments, factor
// evaluation and the two contraction passes of the matvec.
//
// Layout in HBM (N points, leading dimension ldN >= roundup(N, 64) + 64, so
// that vector loads of a row may run up to 63 points past N without leaving
// the row):
//   x_soa : d rows of ldN coordinates (input type), one row per coordinate;
//   phi   : H rows of ldN values, row h = solid harmonic h at every point;
//   q     : S rows of ldN values, row (k,l) = radial function l of degree k.
// Every per-point kernel maps consecutive lanes to consecutive points, so a
// wavefront reads/writes one contiguous 256 B (fp32) or 512 B (fp64) segment
// per row.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <algorithm>
#include <type_traits>

#include "kernels.hpp"

namespace hdf {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef double doublex4 __attribute__((ext_vector_type(4)));

template <typename T> struct Mfma;
// 16x16x4 MFMA.  Operands: lane r + 16 q supplies A[r][q] and B[q][r].
// Accumulator element e of lane j + 16 g holds D[row(g, e)][j]; the row map
// differs between the two instructions (measured on gfx950):
//   f32: row = 4 g + e        f64: row = g + 4 e
template <> struct Mfma<float> {
  typedef floatx4 V;
  static __device__ __forceinline__ V run(float a, float b, V c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int g, int e) { return 4 * g + e; }
};
template <> struct Mfma<double> {
  typedef doublex4 V;
  static __device__ __forceinline__ V run(double a, double b, V c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int g, int e) { return g + 4 * e; }
};

template <typename T> struct Vec2;
template <> struct Vec2<float> { typedef float2 type; };
template <> struct Vec2<double> { typedef double2 type; };

__device__ __forceinline__ double kernel_value_dev(int kind, double r, double l) {
  switch (kind) {
    case 0: return exp(-(r * r) / (2.0 * l * l));
    case 1: return 1.0 / (1.0 + (r * r) / (l * l));
    case 2: { double z = 1.7320508075688772 * r / l; return (1.0 + z) * exp(-z); }
    default: { double z = 2.23606797749979 * r / l; return (1.0 + z + z * z / 3.0) * exp(-z); }
  }
}

// SplitMix64 output number q (1-based) of the stream started at `seed`:
// the generator is counter based, state_q = seed + q * gamma.
__device__ __forceinline__ uint64_t splitmix_at(uint64_t seed, uint64_t q) {
  uint64_t z = seed + q * 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// Fixed-order tree reduction over a 256-thread block (deterministic).
template <typename Op>
__device__ __forceinline__ double block_reduce(double v, double* sh, Op op) {
  const int t = threadIdx.x;
  __syncthreads();
  sh[t] = v;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (t < w) sh[t] = op(sh[t], sh[t + w]);
    __syncthreads();
  }
  return sh[0];
}

struct OpMin { __device__ double operator()(double a, double b) const { return fmin(a, b); } };
struct OpMax { __device__ double operator()(double a, double b) const { return fmax(a, b); } };
struct OpAdd { __device__ double operator()(double a, double b) const { return a + b; } };

// ------------------------------------------------------------------ prep
// Partial record per block: [0..7] min, [8..15] max, [16] nu2, [17] nonfinite.
constexpr int kPrepRec = 18;

// block_reduce of the 18 entries of a prep record at once (entries 0..7 min, 8..15 max, 16..17
// sum): the same fixed tree per entry, with one barrier per level for all of them.
__device__ __forceinline__ void block_reduce_rec(double (&v)[kPrepRec], double (*sh)[256]) {
  const int t = threadIdx.x;
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kPrepRec; ++q) sh[q][t] = v[q];
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (t < w) {
#pragma unroll
      for (int q = 0; q < kPrepRec; ++q) {
        const double a = sh[q][t], b = sh[q][t + w];
        sh[q][t] = q < 8 ? fmin(a, b) : (q < 16 ? fmax(a, b) : a + b);
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int q = 0; q < kPrepRec; ++q) v[q] = sh[q][0];
}

template <typename Tin>
__global__ void __launch_bounds__(256) k_prep_minmax(const Tin* __restrict__ pts, int64_t n, int d,
                                                      int64_t ld, Tin* __restrict__ x_soa,
                                                      int64_t ldx, int kind, double l,
                                                      double* __restrict__ part) {
  __shared__ double shr[kPrepRec][256];
  double mn[8], mx[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) { mn[j] = INFINITY; mx[j] = -INFINITY; }
  double nf = 0.0;
  const int64_t gsz = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gsz) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      if (j < d) {
        const Tin raw = pts[i * ld + j];
        x_soa[(int64_t)j * ldx + i] = raw;
        const double v = (double)raw;
        if (!isfinite(v)) nf += 1.0;
        mn[j] = fmin(mn[j], v);
        mx[j] = fmax(mx[j], v);
      }
    }
  }
  // ||K||_F sample: pair t uses generator outputs 2t+1 and 2t+2
  double nu = 0.0;
  {
#pragma clang fp contract(off)
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < kNuPairs; t += gsz) {
      const uint64_t ia = (splitmix_at(kNuSeed, 2 * (uint64_t)t + 1) >> 11) % (uint64_t)n;
      const uint64_t ib = (splitmix_at(kNuSeed, 2 * (uint64_t)t + 2) >> 11) % (uint64_t)n;
      double s = 0.0;
      for (int j = 0; j < d; ++j) {
        const double df = (double)pts[(int64_t)ia * ld + j] - (double)pts[(int64_t)ib * ld + j];
        s = s + df * df;
      }
      const double kv = kernel_value_dev(kind, sqrt(s), l);
      nu = nu + kv * kv;
    }
  }
  double* rec = part + (int64_t)blockIdx.x * kPrepRec;
  double v[kPrepRec];
#pragma unroll
  for (int j = 0; j < 8; ++j) { v[j] = mn[j]; v[8 + j] = mx[j]; }
  v[16] = nu;
  v[17] = nf;
  block_reduce_rec(v, shr);
  if (threadIdx.x < kPrepRec) {
    double r = v[0];
#pragma unroll
    for (int q = 1; q < kPrepRec; ++q) r = threadIdx.x == q ? v[q] : r;
    rec[threadIdx.x] = r;
  }
}

__global__ void __launch_bounds__(256) k_prep_fin1(const double* __restrict__ part, int nblk,
                                                    GeoDev* geo) {
  __shared__ double shr[kPrepRec][256];
  double v[kPrepRec];
#pragma unroll
  for (int q = 0; q < kPrepRec; ++q) v[q] = (q < 8) ? INFINITY : (q < 16 ? -INFINITY : 0.0);
  for (int b = threadIdx.x; b < nblk; b += 256) {
#pragma unroll
    for (int q = 0; q < kPrepRec; ++q) {
      const double x = part[(int64_t)b * kPrepRec + q];
      v[q] = (q < 8) ? fmin(v[q], x) : (q < 16 ? fmax(v[q], x) : v[q] + x);
    }
  }
  block_reduce_rec(v, shr);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int q = 0; q < 8; ++q) geo->c[q] = (v[q] + v[8 + q]) * 0.5;   // centre of the bounding box
    geo->nu2_sum = v[16];
    geo->nonfinite = v[17];
  }
}

template <typename Tin>
__global__ void __launch_bounds__(256) k_prep_radius(const Tin* __restrict__ x_soa, int64_t ldx,
                                                      int64_t n, int d, const GeoDev* geo,
                                                      double* __restrict__ part) {
#pragma clang fp contract(off)
  __shared__ double sh[256];
  double mx = 0.0;
  const int64_t gsz = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gsz) {
    double s = 0.0;
    for (int j = 0; j < d; ++j) {
      const double t = (double)x_soa[(int64_t)j * ldx + i] - geo->c[j];
      s = s + t * t;
    }
    mx = fmax(mx, s);
  }
  const double r = block_reduce(mx, sh, OpMax());
  if (threadIdx.x == 0) part[blockIdx.x] = r;
}

__global__ void __launch_bounds__(256) k_prep_fin2(const double* __restrict__ part, int nblk,
                                                    GeoDev* geo) {
  __shared__ double sh[256];
  double v = 0.0;
  for (int b = threadIdx.x; b < nblk; b += 256) v = fmax(v, part[b]);
  const double r = block_reduce(v, sh, OpMax());
  if (threadIdx.x == 0) {
    geo->R2 = r;
    geo->R = sqrt(r);
    geo->Reff = geo->R > 0.0 ? geo->R : 1.0;
  }
}

template <typename Tin>
__global__ void __launch_bounds__(256) k_prep_rho(const Tin* __restrict__ x_soa, int64_t ldx,
                                                   int64_t n, int d, const GeoDev* geo,
                                                   double* __restrict__ part) {
#pragma clang fp contract(off)
  __shared__ double sh[256];
  double mn = INFINITY, mx = -INFINITY;
  const double Reff = geo->Reff;
  const int64_t gsz = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gsz) {
    double s = 0.0;
    for (int j = 0; j < d; ++j) {
      const double t = ((double)x_soa[(int64_t)j * ldx + i] - geo->c[j]) / Reff;
      s = s + t * t;
    }
    mn = fmin(mn, s);
    mx = fmax(mx, s);
  }
  const double a = block_reduce(mn, sh, OpMin());
  const double b = block_reduce(mx, sh, OpMax());
  if (threadIdx.x == 0) { part[2 * blockIdx.x] = a; part[2 * blockIdx.x + 1] = b; }
}

__global__ void __launch_bounds__(256) k_prep_fin3(const double* __restrict__ part, int nblk,
                                                    GeoDev* geo) {
  __shared__ double sh[256];
  double mn = INFINITY, mx = -INFINITY;
  for (int b = threadIdx.x; b < nblk; b += 256) {
    mn = fmin(mn, part[2 * b]);
    mx = fmax(mx, part[2 * b + 1]);
  }
  const double a = block_reduce(mn, sh, OpMin());
  const double c = block_reduce(mx, sh, OpMax());
  if (threadIdx.x == 0) { geo->rho2_min = a; geo->rho2_max = c; }
}

hipError_t launch_prep(const void* pts, int dtype, int64_t n, int d, int64_t ld, void* x_soa,
                       int64_t ldx, int kernel, double l, double* partials, GeoDev* geo,
                       hipStream_t s) {
  const int nb = kPrepBlocks;
  if (dtype == 0) {
    k_prep_minmax<float><<<nb, 256, 0, s>>>((const float*)pts, n, d, ld, (float*)x_soa, ldx, kernel, l, partials);
  } else {
    k_prep_minmax<double><<<nb, 256, 0, s>>>((const double*)pts, n, d, ld, (double*)x_soa, ldx, kernel, l, partials);
  }
  k_prep_fin1<<<1, 256, 0, s>>>(partials, nb, geo);
  if (dtype == 0) k_prep_radius<float><<<nb, 256, 0, s>>>((const float*)x_soa, ldx, n, d, geo, partials);
  else k_prep_radius<double><<<nb, 256, 0, s>>>((const double*)x_soa, ldx, n, d, geo, partials);
  k_prep_fin2<<<1, 256, 0, s>>>(partials, nb, geo);
  if (dtype == 0) k_prep_rho<float><<<nb, 256, 0, s>>>((const float*)x_soa, ldx, n, d, geo, partials);
  else k_prep_rho<double><<<nb, 256, 0, s>>>((const double*)x_soa, ldx, n, d, geo, partials);
  k_prep_fin3<<<1, 256, 0, s>>>(partials, nb, geo);
  return hipGetLastError();
}

// Geometry of two point sets (general case X != Y): the existing passes run
// over both sets into adjacent halves of the partial records, so the centre,
// radius and rho^2 interval are those of X u Y.  nu is then replaced by the
// cross-pair estimate: pair t draws generator outputs 2t+1 and 2t+2, a < nx,
// b < ny (the per-set estimates of the min/max pass are discarded).
template <typename Tin>
__global__ void __launch_bounds__(256) k_nu_cross(const Tin* __restrict__ px, int64_t nx, int64_t ldx,
                                                   const Tin* __restrict__ py, int64_t ny, int64_t ldy,
                                                   int d, int kind, double l, double* __restrict__ part) {
  __shared__ double sh[256];
  double nu = 0.0;
  const int64_t gsz = (int64_t)gridDim.x * blockDim.x;
  {
#pragma clang fp contract(off)
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < kNuPairs; t += gsz) {
      const uint64_t ia = (splitmix_at(kNuSeed, 2 * (uint64_t)t + 1) >> 11) % (uint64_t)nx;
      const uint64_t ib = (splitmix_at(kNuSeed, 2 * (uint64_t)t + 2) >> 11) % (uint64_t)ny;
      double s = 0.0;
      for (int j = 0; j < d; ++j) {
        const double df = (double)px[(int64_t)ia * ldx + j] - (double)py[(int64_t)ib * ldy + j];
        s = s + df * df;
      }
      const double kv = kernel_value_dev(kind, sqrt(s), l);
      nu = nu + kv * kv;
    }
  }
  const double r = block_reduce(nu, sh, OpAdd());
  if (threadIdx.x == 0) part[blockIdx.x] = r;
}

__global__ void __launch_bounds__(256) k_nu_fin(const double* __restrict__ part, int nblk, GeoDev* geo) {
  __shared__ double sh[256];
  double v = 0.0;
  for (int b = threadIdx.x; b < nblk; b += 256) v += part[b];
  const double r = block_reduce(v, sh, OpAdd());
  if (threadIdx.x == 0) geo->nu2_sum = r;
}

hipError_t launch_prep_cross(const void* ptsx, int64_t nx, int64_t ldx, const void* ptsy, int64_t ny,
                             int64_t ldy, int dtype, int d, void* soax, int64_t ldsx, void* soay,
                             int64_t ldsy, int kernel, double l, double* partials, GeoDev* geo,
                             hipStream_t s) {
  const int nb = kPrepBlocks;
  double* p1 = partials + (int64_t)nb * kPrepRec;
#define PREP_CROSS(T)                                                                                   \
  k_prep_minmax<T><<<nb, 256, 0, s>>>((const T*)ptsx, nx, d, ldx, (T*)soax, ldsx, kernel, l, partials); \
  k_prep_minmax<T><<<nb, 256, 0, s>>>((const T*)ptsy, ny, d, ldy, (T*)soay, ldsy, kernel, l, p1);       \
  k_prep_fin1<<<1, 256, 0, s>>>(partials, 2 * nb, geo);                                                 \
  k_prep_radius<T><<<nb, 256, 0, s>>>((const T*)soax, ldsx, nx, d, geo, partials);                      \
  k_prep_radius<T><<<nb, 256, 0, s>>>((const T*)soay, ldsy, ny, d, geo, partials + nb);                 \
  k_prep_fin2<<<1, 256, 0, s>>>(partials, 2 * nb, geo);                                                 \
  k_prep_rho<T><<<nb, 256, 0, s>>>((const T*)soax, ldsx, nx, d, geo, partials);                         \
  k_prep_rho<T><<<nb, 256, 0, s>>>((const T*)soay, ldsy, ny, d, geo, partials + 2 * nb);                \
  k_prep_fin3<<<1, 256, 0, s>>>(partials, 2 * nb, geo);                                                 \
  k_nu_cross<T><<<nb, 256, 0, s>>>((const T*)ptsx, nx, ldx, (const T*)ptsy, ny, ldy, d, kernel, l, partials); \
  k_nu_fin<<<1, 256, 0, s>>>(partials, nb, geo);
  if (dtype == 0) {
    PREP_CROSS(float)
  } else {
    PREP_CROSS(double)
  }
#undef PREP_CROSS
  return hipGetLastError();
}

// ------------------------------------------------------------------ sampled pairs
template <typename Tin>
__global__ void __launch_bounds__(256) k_pairs(const Tin* __restrict__ x_soa, int64_t ldx, int64_t n, int d,
                                                const GeoDev* __restrict__ geo, uint64_t seed, int M,
                                                double* __restrict__ out, int32_t* __restrict__ idx) {
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t >= M) return;
  const int64_t a = (int64_t)((splitmix_at(seed, 2 * (uint64_t)t + 1) >> 11) % (uint64_t)n);
  const int64_t b = (int64_t)((splitmix_at(seed, 2 * (uint64_t)t + 2) >> 11) % (uint64_t)n);
  const double Reff = geo->Reff;
  double r2 = 0.0, ra2 = 0.0, rb2 = 0.0, dot = 0.0;
  for (int j = 0; j < d; ++j) {
    const double xa = (double)x_soa[(int64_t)j * ldx + a], xb = (double)x_soa[(int64_t)j * ldx + b];
    const double df = xa - xb;
    const double ua = (xa - geo->c[j]) / Reff, ub = (xb - geo->c[j]) / Reff;
    r2 += df * df;
    ra2 += ua * ua;
    rb2 += ub * ub;
    dot += ua * ub;
  }
  out[t] = sqrt(r2);
  out[M + t] = ra2;
  out[2 * M + t] = rb2;
  out[3 * M + t] = dot;
  idx[t] = (int32_t)a;
  idx[M + t] = (int32_t)b;
}

hipError_t launch_pairs(const void* x_soa, int dtype, int64_t ldx, int64_t n, int d, const GeoDev* geo,
                        uint64_t seed, int M, double* out, int32_t* idx, hipStream_t s) {
  if (M <= 0) return hipSuccess;
  const unsigned nb = (unsigned)((M + 255) / 256);
  if (dtype == 0) k_pairs<float><<<nb, 256, 0, s>>>((const float*)x_soa, ldx, n, d, geo, seed, M, out, idx);
  else k_pairs<double><<<nb, 256, 0, s>>>((const double*)x_soa, ldx, n, d, geo, seed, M, out, idx);
  return hipGetLastError();
}

// ------------------------------------------------------------------ Gram
// Moments mu[k][c] = sum_i rho_i^{2k} T_c(t_i) as a tall-skinny product
// A^T B on MFMA (A[i][k] = rho_i^{2k}, B[i][c] = T_c(t_i)).  The per-degree
// Gram blocks follow on the host from T_a T_b = (T_{a+b} + T_{|a-b|}) / 2.
constexpr int kGramRowTiles = 2;   // k <= 31
constexpr int kGramColTiles = 4;   // c <= 63
constexpr int kGramWaves = 4096;   // target wavefronts per Gram launch

// Per-point radial variables: rho^2 = ||(x - c)/R||^2 and the Chebyshev
// argument t of the radial basis.
template <typename Tin>
__device__ __forceinline__ void radial_point(const Tin* __restrict__ x_soa, int64_t ldx, int64_t i,
                                             int d, const GeoDev* __restrict__ geo, double Reff,
                                             double u0, double u1, double& rho2, double& t) {
  double s = 0.0;
  for (int j = 0; j < d; ++j) {
    const double v = ((double)x_soa[(int64_t)j * ldx + i] - geo->c[j]) / Reff;
    s += v * v;
  }
  rho2 = s;
  t = (2.0 * s - u0 - u1) / (u1 - u0);
}

// A wavefront of the Gram passes takes chunks of `tpc` tiles of 16 points: lane p < 16 tpc evaluates the
// radial variables of the chunk's point p (a division per coordinate, the longest part of a tile) once
// and leaves them in LDS for the lanes that use them.  Chunks of four tiles keep all lanes busy with it;
// where that would leave wavefronts of the launch without a chunk, chunks of one.  Evaluated by each
// lane that used them, k_gram2 took 351 us on 200,000 points in d = 4 (thirteen degrees) and 156 so; in
// one of sixteen lanes for a tile, k_gram 99 us on 1e6 points in d = 5 and 86 so.
static int gram_chunk_tiles(int64_t n, int64_t waves) { return (n + 63) / 64 >= waves ? 4 : 1; }

// A 16-point tile feeds four MFMA K-steps: in step e, lane group g (lanes
// 16g..16g+15) supplies point tile*16 + g + 4e, lane r of the group supplies
// row / column index r of the two operands.  Any bijection between (g, e)
// and the 16 points is valid because the points are summed over.
// NRT x NCT moment tiles (rows k < 16 NRT, columns c < 16 NCT) are compile-time
// sizes, so the accumulators of unused tiles take no registers.
template <typename Tin, int MODE, int NRT, int NCT>
__global__ void __launch_bounds__(256) k_gram(const Tin* __restrict__ x_soa, int64_t ldx, int64_t n,
                                               int d, const GeoDev* __restrict__ geo, double u0,
                                               double u1, int K, int tpc, double* __restrict__ part) {
  constexpr int nrt = NRT, nct = NCT;
  typedef typename std::conditional<MODE == 0, double, float>::type T;
  typedef typename Mfma<T>::V V;
  __shared__ double sh[4][4 * 64];
  // T_c(t) (c < 16 NCT) and rho^2 of a tile's 16 points, one row per point, per wavefront
  constexpr int TCS = 16 * NCT + 1;
  __shared__ double tcs[4][16 * TCS];
  __shared__ double rad[4][2 * 64];                 // rho^2 and t of the chunk's points
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int li = lane & 15, g = lane >> 4;
  const double Reff = geo->Reff;
  double dacc[NRT][NCT][4];
#pragma unroll
  for (int a = 0; a < NRT; ++a)
#pragma unroll
    for (int b = 0; b < NCT; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) dacc[a][b][e] = 0.0;
  const int64_t ntile = (n + 15) / 16;
  int since_flush = 0;
  V acc[NRT][NCT];
#pragma unroll
  for (int a = 0; a < NRT; ++a)
#pragma unroll
    for (int b = 0; b < NCT; ++b) acc[a][b] = V{0, 0, 0, 0};
  const int64_t tiles_step = (int64_t)gridDim.x * 4 * tpc;
  for (int64_t tile0 = ((int64_t)blockIdx.x * 4 + wave) * tpc; tile0 < ntile; tile0 += tiles_step) {
    if (lane < 16 * tpc) {
      const int64_t i = tile0 * 16 + lane;
      double rho2 = 0.0, tp = 0.0;
      if (i < n) radial_point(x_soa, ldx, i, d, geo, Reff, u0, u1, rho2, tp);
      rad[wave][lane] = rho2;
      rad[wave][64 + lane] = tp;
    }
    __builtin_amdgcn_wave_barrier();
    for (int tt = 0; tt < tpc; ++tt) {
      const int64_t tile = tile0 + tt;
      if (tile >= ntile) break;                       // uniform
      double w[NRT][4], tc[NCT][4];
      // the T_c(t) recurrence of point g + 4 e runs once, in lane e of group g, and goes through LDS to
      // the sixteen lanes that use it (T_c for c = b*16 + li, rho^2 for the powers rho^(2k),
      // k = a*16 + li)
      double* trow = &tcs[wave][0];
      if (li < 4) {
        const double rho2 = rad[wave][16 * tt + g + 4 * li], tp = rad[wave][64 + 16 * tt + g + 4 * li];
        double* dst = trow + (g + 4 * li) * TCS;
        dst[16 * NCT] = rho2;
        double tm1 = 1.0, t0 = tp;
#pragma unroll
        for (int c = 0; c < 16 * NCT; ++c) {
          double cur;
          if (c == 0) cur = 1.0;
          else if (c == 1) cur = tp;
          else { cur = 2.0 * tp * t0 - tm1; tm1 = t0; t0 = cur; }
          dst[c] = cur;
        }
      }
      // the rows are read by the other lanes of the wavefront (wavefront-synchronous exchange; the
      // next tile's rows are written after this tile's MFMAs, which every lane reaches first)
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int64_t i = tile * 16 + g + 4 * e;
        const double rho2 = trow[(g + 4 * e) * TCS + 16 * NCT];
#pragma unroll
        for (int a = 0; a < NRT; ++a) {
          const int k = a * 16 + li;
          double pw = 0.0;
          if (i < n && a < nrt && k <= K) {
            pw = 1.0;
            double base = rho2;
            for (int q = k; q > 0; q >>= 1) {
              if (q & 1) pw *= base;
              base *= base;
            }
          }
          w[a][e] = pw;
        }
      }
#pragma unroll
      for (int b = 0; b < NCT; ++b) {
        const int c = b * 16 + li;
#pragma unroll
        for (int e = 0; e < 4; ++e) tc[b][e] = (b < nct && c <= 2 * K) ? trow[(g + 4 * e) * TCS + c] : 0.0;
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int64_t i = tile * 16 + g + 4 * e;
#pragma unroll
        for (int a = 0; a < NRT; ++a) {
          if (a >= nrt) continue;
#pragma unroll
          for (int b = 0; b < NCT; ++b) {
            if (b >= nct) continue;
            const double wv = (i < n) ? w[a][e] : 0.0;
            if constexpr (MODE == 2) {
              const float ah = (float)wv, al = (float)(wv - (double)ah);
              const float bh = (float)tc[b][e], bl = (float)(tc[b][e] - (double)bh);
              acc[a][b] = Mfma<float>::run(ah, bh, acc[a][b]);
              acc[a][b] = Mfma<float>::run(ah, bl, acc[a][b]);
              acc[a][b] = Mfma<float>::run(al, bh, acc[a][b]);
            } else {
              acc[a][b] = Mfma<T>::run((T)wv, (T)tc[b][e], acc[a][b]);
            }
          }
        }
      }
      // binary32 accumulators are flushed to binary64 every 4 tiles (64 points)
      if (MODE != 0 && ++since_flush == 4) {
        since_flush = 0;
#pragma unroll
        for (int a = 0; a < NRT; ++a)
#pragma unroll
          for (int b = 0; b < NCT; ++b) {
#pragma unroll
            for (int e = 0; e < 4; ++e) dacc[a][b][e] += (double)acc[a][b][e];
            acc[a][b] = V{0, 0, 0, 0};
          }
      }
    }
  }
#pragma unroll
  for (int a = 0; a < NRT; ++a)
#pragma unroll
    for (int b = 0; b < NCT; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) dacc[a][b][e] += (double)acc[a][b][e];
  // combine the four waves in a fixed order, one 16x16 tile at a time
  const int rows = nrt * 16, cols = nct * 16;
  double* out = part + (int64_t)blockIdx.x * rows * cols;
#pragma unroll
  for (int a = 0; a < NRT; ++a)
#pragma unroll
    for (int b = 0; b < NCT; ++b) {
      if (a >= nrt || b >= nct) continue;
      __syncthreads();
#pragma unroll
      for (int e = 0; e < 4; ++e) sh[wave][e * 64 + lane] = dacc[a][b][e];
      __syncthreads();
      const int idx = threadIdx.x;             // 256 = 4 elements x 64 lanes
      const int ln = idx & 63, e = idx >> 6;
      const double v = sh[0][idx] + sh[1][idx] + sh[2][idx] + sh[3][idx];
      const int row = a * 16 + Mfma<T>::row(ln >> 4, e), col = b * 16 + (ln & 15);
      out[row * cols + col] = v;
    }
}

// Fixed-order sum of the per-block partial records, out[e] = sum_b part[b][e].
// A block owns 64 consecutive entries; wavefront w takes the records b = w, w + 16, ... with eight
// independent running sums (loads in flight), and the sixteen wavefront sums are combined in a fixed
// order through LDS.  A few blocks (512 entries make eight) read 1,024 records: the chain of loads of a
// wavefront is what takes the time.
constexpr int kFinWaves = 16;

__global__ void __launch_bounds__(64 * kFinWaves) k_gram_fin(const double* __restrict__ part, int nblk, int total,
                                                             double* __restrict__ out) {
  __shared__ double red[kFinWaves][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int e = blockIdx.x * 64 + lane;
  const int ee = e < total ? e : 0;
  double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  int b = w;
  for (; b + 7 * kFinWaves < nblk; b += 8 * kFinWaves)
#pragma unroll
    for (int u = 0; u < 8; ++u) acc[u] += part[(int64_t)(b + kFinWaves * u) * total + ee];
  for (; b < nblk; b += kFinWaves) acc[0] += part[(int64_t)b * total + ee];
  red[w][lane] = ((acc[0] + acc[1]) + (acc[2] + acc[3])) + ((acc[4] + acc[5]) + (acc[6] + acc[7]));
  __syncthreads();
  if (w == 0 && e < total) {
    double t = 0.0;
    for (int v = 0; v < kFinWaves; ++v) t += red[v][lane];
    out[e] = t;
  }
}

int gram_blocks(int64_t n) {
  const int64_t tiles = (n + 15) / 16;
  int64_t b = (tiles + 3) / 4;
  if (b > kGramWaves / 4) b = kGramWaves / 4;
  if (b < 1) b = 1;
  return (int)b;
}

hipError_t launch_gram(const void* x_soa, int dtype, int64_t ldx, int64_t n, int d,
                       const GeoDev* geo, double u0, double u1, int K, int mode,
                       double* partials, double* moments, hipStream_t s) {
  const int nrt = (K + 1 + 15) / 16, nct = (2 * K + 1 + 15) / 16;
  if (nrt > kGramRowTiles || nct > kGramColTiles) return hipErrorInvalidValue;
  const int nb = gram_blocks(n), tpc = gram_chunk_tiles(n, 4 * nb);
#define GRAM_TILES(TIN, MODE, R, C)                                                               \
  k_gram<TIN, MODE, R, C><<<nb, 256, 0, s>>>((const TIN*)x_soa, ldx, n, d, geo, u0, u1, K, tpc, partials)
#define GRAM_LAUNCH(TIN, MODE)                                                                    \
  do {                                                                                            \
    if (nrt == 1 && nct == 1) GRAM_TILES(TIN, MODE, 1, 1);                                         \
    else if (nrt == 1 && nct == 2) GRAM_TILES(TIN, MODE, 1, 2);                                    \
    else if (nrt == 2 && nct == 3) GRAM_TILES(TIN, MODE, 2, 3);                                    \
    else if (nrt == 2 && nct == 4) GRAM_TILES(TIN, MODE, 2, 4);                                    \
    else return hipErrorInvalidValue;                                                             \
  } while (0)
  if (dtype == 0) {
    if (mode == 0) GRAM_LAUNCH(float, 0);
    else if (mode == 1) GRAM_LAUNCH(float, 1);
    else GRAM_LAUNCH(float, 2);
  } else {
    if (mode == 0) GRAM_LAUNCH(double, 0);
    else if (mode == 1) GRAM_LAUNCH(double, 1);
    else GRAM_LAUNCH(double, 2);
  }
#undef GRAM_LAUNCH
#undef GRAM_TILES
  const int total = nrt * 16 * nct * 16;
  k_gram_fin<<<(total + 63) / 64, 64 * kFinWaves, 0, s>>>(partials, nb, total, moments);
  return hipGetLastError();
}

// Second Gram pass (refinement of the compression, binary64 MFMA): for degree
// k = blockIdx.y, G2_k = sum_i z_i z_i^T with z_i = T1_k^T y_i and
// y_i[a] = rho_i^k T_a(t_i), a < L_k = K - k + 1.  T1_k (L_k x L_k, row-major)
// is the preconditioner from the first pass, so the columns Y_k T1_k are
// nearly orthonormal and their Gram is accurate in binary64 even when Y_k is
// badly conditioned.  z is formed on the VALU (lane r of group g holds z_r
// and z_{16+r} of four points), then accumulated as z z^T on MFMA with the
// same (g, e) -> point bijection as the first pass.  Partial record per
// block and degree: [32][32].
template <typename Tin>
__global__ void __launch_bounds__(256) k_gram2(const Tin* __restrict__ x_soa, int64_t ldx, int64_t n,
                                                int d, const GeoDev* __restrict__ geo, double u0,
                                                double u1, int K, int tpc, const double* __restrict__ T1,
                                                const int32_t* __restrict__ t1_off,
                                                const int32_t* __restrict__ sel, int n_sel,
                                                double* __restrict__ part) {
  typedef Mfma<double>::V V;
  __shared__ double t1s[32 * 32];
  __shared__ double sh[4][4 * 64];
  __shared__ double rad[4][2 * 64];                 // t and rho^k of the chunk's points
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int li = lane & 15, g = lane >> 4;
  const int k = sel[blockIdx.y];
  const int L = K - k + 1;
  const int nt = (L + 15) / 16;
  const double Reff = geo->Reff;
  for (int e = threadIdx.x; e < L * L; e += 256) t1s[e] = T1[t1_off[k] + e];
  __syncthreads();
  V acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[a][b] = V{0, 0, 0, 0};
  const bool j0 = li < L, j1 = 16 + li < L;
  const int64_t ntile = (n + 15) / 16;
  const int64_t tiles_step = (int64_t)gridDim.x * 4 * tpc;
  for (int64_t tile0 = ((int64_t)blockIdx.x * 4 + wave) * tpc; tile0 < ntile; tile0 += tiles_step) {
    if (lane < 16 * tpc) {
      const int64_t i = tile0 * 16 + lane;
      double rho2 = 0.0, tp = 0.0, pw = 0.0;
      if (i < n) {
        radial_point(x_soa, ldx, i, d, geo, Reff, u0, u1, rho2, tp);
        pw = 1.0;
        double base = sqrt(rho2);
        for (int q = k; q > 0; q >>= 1) {
          if (q & 1) pw *= base;
          base *= base;
        }
      }
      rad[wave][lane] = tp;
      rad[wave][64 + lane] = pw;
    }
    __builtin_amdgcn_wave_barrier();
    for (int tt = 0; tt < tpc; ++tt) {
      if (tile0 + tt >= ntile) break;                 // uniform
      double t[4], rk[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        t[e] = rad[wave][16 * tt + g + 4 * e];
        rk[e] = rad[wave][64 + 16 * tt + g + 4 * e];
      }
      double z0[4] = {0, 0, 0, 0}, z1[4] = {0, 0, 0, 0};
      double tm1[4], tc[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) { tm1[e] = 0.0; tc[e] = 1.0; }
      for (int a = 0; a < L; ++a) {
        const double c0 = j0 ? t1s[a * L + li] : 0.0;
        const double c1 = j1 ? t1s[a * L + 16 + li] : 0.0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (a == 1) { tm1[e] = 1.0; tc[e] = t[e]; }
          else if (a >= 2) { const double tn = 2.0 * t[e] * tc[e] - tm1[e]; tm1[e] = tc[e]; tc[e] = tn; }
          const double ya = rk[e] * tc[e];
          z0[e] += c0 * ya;
          if (nt > 1) z1[e] += c1 * ya;               // uniform
        }
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        acc[0][0] = Mfma<double>::run(z0[e], z0[e], acc[0][0]);
        if (nt > 1) {
          acc[0][1] = Mfma<double>::run(z0[e], z1[e], acc[0][1]);
          acc[1][0] = Mfma<double>::run(z1[e], z0[e], acc[1][0]);
          acc[1][1] = Mfma<double>::run(z1[e], z1[e], acc[1][1]);
        }
      }
    }
  }
  double* out = part + ((int64_t)blockIdx.x * n_sel + blockIdx.y) * 1024;
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      if (a >= nt || b >= nt) continue;
      __syncthreads();
#pragma unroll
      for (int e = 0; e < 4; ++e) sh[wave][e * 64 + lane] = acc[a][b][e];
      __syncthreads();
      const int idx = threadIdx.x, ln = idx & 63, e = idx >> 6;
      const double v = sh[0][idx] + sh[1][idx] + sh[2][idx] + sh[3][idx];
      const int row = a * 16 + Mfma<double>::row(ln >> 4, e), col = b * 16 + (ln & 15);
      out[row * 32 + col] = v;
    }
}

int gram2_blocks(int64_t n, int n_sel) {
  const int64_t tiles = (n + 15) / 16;
  int64_t b = (tiles + 3) / 4;
  const int64_t cap = std::max<int64_t>(1, kGramWaves / (4 * n_sel));
  if (b > cap) b = cap;
  if (b < 1) b = 1;
  return (int)b;
}

hipError_t launch_gram2(const void* x_soa, int dtype, int64_t ldx, int64_t n, int d,
                        const GeoDev* geo, double u0, double u1, int K, const double* T1,
                        const int32_t* t1_off, const int32_t* sel, int n_sel, double* partials,
                        double* out, hipStream_t s) {
  if (K + 1 > 32 || n_sel < 1) return hipErrorInvalidValue;
  const int nb = gram2_blocks(n, n_sel), tpc = gram_chunk_tiles(n, 4 * nb);
  const dim3 grid(nb, n_sel);
  if (dtype == 0)
    k_gram2<float><<<grid, 256, 0, s>>>((const float*)x_soa, ldx, n, d, geo, u0, u1, K, tpc, T1, t1_off, sel,
                                        n_sel, partials);
  else
    k_gram2<double><<<grid, 256, 0, s>>>((const double*)x_soa, ldx, n, d, geo, u0, u1, K, tpc, T1, t1_off, sel,
                                         n_sel, partials);
  const int total = n_sel * 1024;
  k_gram_fin<<<(total + 63) / 64, 64 * kFinWaves, 0, s>>>(partials, nb, total, out);
  return hipGetLastError();
}

// ------------------------------------------------------------------ build
// Solid harmonics by nested normalised Gegenbauer chain recurrences.  The
// loops run from the innermost chain level outwards (azimuthal index first,
// degree k last), so each level keeps only its two-term recurrence state in
// registers; every iteration of the innermost loop yields one harmonic,
// stored to its canonical row col_of[t] (the table follows this loop order).
// Each thread evaluates PPT consecutive points (independent recurrence chains
// in flight) and writes them with one 16-byte nontemporal store per row.
typedef double doublex2 __attribute__((ext_vector_type(2)));
template <typename T, int PPT> struct PVec;
template <> struct PVec<float, 4> { typedef floatx4 type; };
template <> struct PVec<double, 2> { typedef doublex2 type; };

template <typename T, int PPT>
__device__ __forceinline__ void store_row(T* __restrict__ dst, const T (&v)[PPT]) {
  typedef typename PVec<T, PPT>::type V;
  V w;
#pragma unroll
  for (int e = 0; e < PPT; ++e) w[e] = v[e];
  __builtin_nontemporal_store(w, reinterpret_cast<V*>(dst));
}

// SPLIT: only the harmonics of loop order [t_lo, t_hi) are evaluated; a subtree outside the range is
// passed over by its number of harmonics, leaves[level (K + 1) + b] below a level-`level` loop of base b.
template <typename T, int D, int PPT, int LEVEL, bool SPLIT>
struct Chain {
  typedef typename Vec2<T>::type T2;
  static __device__ __forceinline__ void run(const T (&xt)[PPT][D], const T (&r2)[PPT][D], int b,
                                             const T (&prefix)[PPT], int K,
                                             const T2* __restrict__ chain,
                                             const int32_t* __restrict__ col_of,
                                             const int32_t* __restrict__ leaves, int t_lo, int t_hi, int& t,
                                             T* __restrict__ phi_base, int64_t ld) {
    const T2* cf = chain + ((int64_t)(LEVEL - 1) * (K + 1) + b) * (K + 1);
    T pm1[PPT], p[PPT], pre[PPT];
#pragma unroll
    for (int e = 0; e < PPT; ++e) { pm1[e] = 0; p[e] = cf[0].x; }
    for (int nn = 0; nn <= K - b; ++nn) {
      if (nn == 1) {
#pragma unroll
        for (int e = 0; e < PPT; ++e) { pm1[e] = p[e]; p[e] = cf[1].x * xt[e][LEVEL - 1]; }
      } else if (nn >= 2) {
        const T A = cf[nn].x, B = cf[nn].y;
#pragma unroll
        for (int e = 0; e < PPT; ++e) {
          const T pn = A * xt[e][LEVEL - 1] * p[e] - B * r2[e][LEVEL - 1] * pm1[e];
          pm1[e] = p[e];
          p[e] = pn;
        }
      }
      if constexpr (SPLIT) {
        const int cnt = leaves[(LEVEL - 1) * (K + 1) + b + nn];
        if (t >= t_hi) return;
        if (t + cnt <= t_lo) {
          t += cnt;
          continue;
        }
      }
#pragma unroll
      for (int e = 0; e < PPT; ++e) pre[e] = prefix[e] * p[e];
      Chain<T, D, PPT, LEVEL - 1, SPLIT>::run(xt, r2, b + nn, pre, K, chain, col_of, leaves, t_lo, t_hi, t, phi_base,
                                              ld);
    }
  }
};
template <typename T, int D, int PPT, bool SPLIT>
struct Chain<T, D, PPT, 0, SPLIT> {
  typedef typename Vec2<T>::type T2;
  static __device__ __forceinline__ void run(const T (&)[PPT][D], const T (&)[PPT][D], int,
                                             const T (&prefix)[PPT], int, const T2* __restrict__,
                                             const int32_t* __restrict__ col_of, const int32_t* __restrict__, int, int,
                                             int& t, T* __restrict__ phi_base, int64_t ld) {
    const int col = col_of[t++];
    if (col >= 0) store_row<T, PPT>(phi_base + (int64_t)col * ld, prefix);
  }
};

// Points of a row that the evaluation writes: the n points and zeros up to the padding the streaming
// kernels may read (rows are at least that long).
__host__ __device__ static inline int64_t row_end(int64_t n) { return (n + 63) / 64 * 64 + 64; }

template <typename Tin, typename T, int D, int PPT, bool SPLIT>
__global__ void __launch_bounds__(256) k_build(const Tin* __restrict__ x_soa, int64_t ldx, int64_t n,
                                                const GeoDev* __restrict__ geo, double u0, double u1,
                                                const int32_t* __restrict__ col_of,
                                                const typename Vec2<T>::type* __restrict__ chain,
                                                const int32_t* __restrict__ q_len,
                                                const int32_t* __restrict__ q_off,
                                                const T* __restrict__ q_coef, int K, int S,
                                                const int32_t* __restrict__ leaves, int per_group, int q_per_group,
                                                T* __restrict__ phi, int64_t ld_phi,
                                                T* __restrict__ q, int64_t ld_q) {
  const int64_t i0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * PPT;
  if (i0 >= row_end(n)) return;      // whole thread past the row's written end (a multiple of 64)
  // SPLIT: this workgroup's harmonics (loop order) and radial rows
  const int t_lo = SPLIT ? (int)blockIdx.y * per_group : 0, t_hi = SPLIT ? t_lo + per_group : 0;
  const int q_lo = SPLIT ? (int)blockIdx.y * q_per_group : 0;
  const int q_hi = SPLIT ? (q_lo + q_per_group < S ? q_lo + q_per_group : S) : S;
  T xt[PPT][D], r2[PPT][D], tt[PPT];
  {
#pragma clang fp contract(off)
    const double Reff = geo->Reff;
#pragma unroll
    for (int e = 0; e < PPT; ++e) {
      const int64_t i = (i0 + e < n) ? i0 + e : n - 1;
      double rho2 = 0.0;
#pragma unroll
      for (int j = 0; j < D; ++j) {
        const double v = ((double)x_soa[(int64_t)j * ldx + i] - geo->c[j]) / Reff;
        xt[e][j] = (T)v;
        rho2 = rho2 + v * v;
      }
      tt[e] = (T)((2.0 * rho2 - u0 - u1) / (u1 - u0));
    }
  }
#pragma unroll
  for (int e = 0; e < PPT; ++e) {
    T acc = 0;
#pragma unroll
    for (int j = D - 1; j >= 0; --j) {
      acc += xt[e][j] * xt[e][j];
      r2[e][j] = acc;
    }
  }
  // harmonics: azimuthal part (x_{D-1} + i x_D)^m outermost
  int t = 0;
  T cr[PPT], ci[PPT], pre[PPT];
#pragma unroll
  for (int e = 0; e < PPT; ++e) { cr[e] = i0 + e < n ? 1 : 0; ci[e] = 0; }   // points past n: zero rows
  const T inv_sqrt_2pi = (T)0.39894228040143267794, inv_sqrt_pi = (T)0.56418958354775628695;
  T* phi_base = phi + i0;
  for (int mm = 0; mm <= K; ++mm) {
    if (mm > 0) {
#pragma unroll
      for (int e = 0; e < PPT; ++e) {
        const T ax = xt[e][D - 2], ay = xt[e][D - 1];
        const T ncr = ax * cr[e] - ay * ci[e];
        ci[e] = ay * cr[e] + ax * ci[e];
        cr[e] = ncr;
      }
    }
    const T cm = (mm == 0) ? inv_sqrt_2pi : inv_sqrt_pi;
    if constexpr (SPLIT) {
      if (t >= t_hi) break;
      const int both = (mm > 0 ? 2 : 1) * leaves[(D - 2) * (K + 1) + mm];
      if (t + both <= t_lo) {
        t += both;
        continue;
      }
    }
#pragma unroll
    for (int e = 0; e < PPT; ++e) pre[e] = cm * cr[e];
    Chain<T, D, PPT, D - 2, SPLIT>::run(xt, r2, mm, pre, K, chain, col_of, leaves, t_lo, t_hi, t, phi_base, ld_phi);
    if (mm > 0) {
#pragma unroll
      for (int e = 0; e < PPT; ++e) pre[e] = cm * ci[e];
      Chain<T, D, PPT, D - 2, SPLIT>::run(xt, r2, mm, pre, K, chain, col_of, leaves, t_lo, t_hi, t, phi_base, ld_phi);
    }
  }
  // radial functions: Clenshaw in the basis T_a(t)
  for (int row = q_lo; row < q_hi; ++row) {
    const int L = q_len[row];
    const T* cf = q_coef + q_off[row];
    T b1[PPT], b2[PPT], val[PPT];
#pragma unroll
    for (int e = 0; e < PPT; ++e) { b1[e] = 0; b2[e] = 0; }
    for (int a = L - 1; a >= 1; --a) {
      const T c = cf[a];
#pragma unroll
      for (int e = 0; e < PPT; ++e) {
        const T b0 = 2 * tt[e] * b1[e] - b2[e] + c;
        b2[e] = b1[e];
        b1[e] = b0;
      }
    }
#pragma unroll
    for (int e = 0; e < PPT; ++e) val[e] = i0 + e < n ? tt[e] * b1[e] - b2[e] + cf[0] : (T)0;
    store_row<T, PPT>(q + (int64_t)row * ld_q + i0, val);
  }
}

// Workgroups of the factor evaluation.  One workgroup per 256 PPT points leaves the chip idle for few
// points (10 workgroups for 10,007 points) and, since a thread then writes all its rows one after the
// other, keeps too few stores in flight for many: the harmonics (loop order) and radial rows are cut
// into groups, 16 harmonics or more each, for about kBuildBlocks workgroups in all.  Where that leaves
// fewer than kBuildFewBlocks, groups go down to two harmonics: the chain of a thread is then shorter
// than the recurrences that it repeats.  Kernel times before and now: 2,000 points d = 3 binary64 26 ->
// 7.7 us; 460 points d = 8 binary64 530 -> 14; 10,007 points d = 5 365 -> 24; 1e5 points d = 3 98 -> 27;
// 2e5 points d = 4 316 -> 177; 250,007 points d = 5 binary64 521 -> 473; 1e6 points d = 5 732 -> 687
// (655 at best, 5.2 TB/s).  16,384 workgroups: 1e6 points 760 us, 2e5 points 206; 1,024: 711 and 215.
constexpr int64_t kBuildBlocks = 8192, kBuildFewBlocks = 512;

template <typename Tin, typename T>
static hipError_t launch_build_t(const void* x_soa, int64_t ldx, int64_t n, int d, const GeoDev* geo,
                                 double u0, double u1, const BuildTables& tb, void* phi,
                                 int64_t ld_phi, void* q, int64_t ld_q, hipStream_t s) {
  constexpr int PPT = 16 / sizeof(T);
  if (ld_phi < row_end(n) || ld_q < row_end(n)) return hipErrorInvalidValue;
  const int64_t blocks = (row_end(n) + 256 * PPT - 1) / (256 * PPT);
  const int64_t full = std::min<int64_t>((kBuildBlocks + blocks - 1) / blocks, (tb.n_loop + 15) / 16);
  const int64_t few = std::min<int64_t>((kBuildFewBlocks + blocks - 1) / blocks, (tb.n_loop + 1) / 2);
  const int groups = (int)std::max<int64_t>(1, std::max(full, few));
  const int per_group = (tb.n_loop + groups - 1) / groups, q_per_group = (tb.S + groups - 1) / groups;
  const dim3 grid((unsigned)blocks, (unsigned)groups);
  typedef typename Vec2<T>::type T2;
#define BUILD_RUN(DD, SPLIT)                                                                  \
  k_build<Tin, T, DD, PPT, SPLIT><<<grid, 256, 0, s>>>((const Tin*)x_soa, ldx, n, geo, u0, u1, tb.col_of,       \
                                                       (const T2*)tb.chain, tb.q_len, tb.q_off,                 \
                                                       (const T*)tb.q_coef, tb.K, tb.S, tb.leaves, per_group,   \
                                                       q_per_group, (T*)phi, ld_phi, (T*)q, ld_q)
#define BUILD_CASE(DD)                                                                        \
  case DD:                                                                                    \
    if (groups > 1) BUILD_RUN(DD, true);                                                      \
    else BUILD_RUN(DD, false);                                                                \
    break;
  switch (d) {
    BUILD_CASE(3)
    BUILD_CASE(4)
    BUILD_CASE(5)
    BUILD_CASE(6)
    BUILD_CASE(7)
    BUILD_CASE(8)
    default: return hipErrorInvalidValue;
  }
#undef BUILD_CASE
#undef BUILD_RUN
  return hipGetLastError();
}

hipError_t launch_build(const void* x_soa, int dtype, int64_t ldx, int64_t n, int d,
                        const GeoDev* geo, double u0, double u1, const BuildTables& tb,
                        int prec, void* phi, int64_t ld_phi, void* q, int64_t ld_q,
                        hipStream_t s) {
  if (prec == 1 && dtype == 0)
    return launch_build_t<float, float>(x_soa, ldx, n, d, geo, u0, u1, tb, phi, ld_phi, q, ld_q, s);
  if (prec == 0 && dtype == 1)
    return launch_build_t<double, double>(x_soa, ldx, n, d, geo, u0, u1, tb, phi, ld_phi, q, ld_q, s);
  if (prec == 0 && dtype == 0)        // binary64 factor of binary32 points (tolerances below binary32)
    return launch_build_t<float, double>(x_soa, ldx, n, d, geo, u0, u1, tb, phi, ld_phi, q, ld_q, s);
  return hipErrorInvalidValue;
}

// ------------------------------------------------------------------ adjoint
// dF/dx_i for F = sum_c w_c^T U C U^T v_c, C = diag(lambda) (structure frozen), with
// U[i,(k,h,l)] = S_h(xt_i) q_{k,l}(rho_i^2), xt = (x - c)/R:
//   dF/dx_i = (1/R) sum_{k,h} [ a_h(i) grad S_h(xt_i) + 2 xt_i b_h(i) S_h(xt_i) ],
//   a_h = sum_l q_{k,l} alpha_{h,l},  b_h = sum_l q'_{k,l} alpha_{h,l},
//   alpha_{h,l}(i) = sum_c w_ic Gv[(k,h,l)][c] + v_ic Gw[(k,h,l)][c],  Gv = C U^T V, Gw = C U^T W.
// Both terms are factor contractions: the second is the product of U' (q replaced by q' =
// dq/d(rho^2)) with [Gv | Gw]; the first, since every partial derivative of a degree-k solid
// harmonic is a combination of the degree k-1 ones (dS_{k,h}/dx_j = sum_h' G_k^(j)[h][h'] S_{k-1,h'}),
// is the product of the shifted factor S_{k-1,h'} q_{k,l} with [G^(j)T Gv | G^(j)T Gw] for every j.
// The contractions run through the pass-2 kernel; k_radial evaluates q', k_adj_combine adds up.

// out[row][i] = scale * sum_{a < len} coef[a] T_a(t_i) for the S rows of a coefficient table (the
// radial-function tables with derivative coefficients give q' = dq/d(rho^2)); PPT points per thread.
template <typename Tin, typename T, int PPT>
__global__ void __launch_bounds__(256) k_radial(const Tin* __restrict__ x_soa, int64_t ldx, int64_t n, int d,
                                                 const GeoDev* __restrict__ geo, double u0, double u1,
                                                 const int32_t* __restrict__ q_len, const int32_t* __restrict__ q_off,
                                                 const T* __restrict__ coef, int S, T scale, T* __restrict__ out,
                                                 int64_t ld_out) {
  const int64_t i0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * PPT;
  if (i0 >= row_end(n)) return;      // whole thread past the row's written end (a multiple of 64)
  T tt[PPT];
  {
#pragma clang fp contract(off)
    const double Reff = geo->Reff;
#pragma unroll
    for (int e = 0; e < PPT; ++e) {
      const int64_t i = (i0 + e < n) ? i0 + e : n - 1;
      double rho2 = 0.0;
      for (int j = 0; j < d; ++j) {
        const double v = ((double)x_soa[(int64_t)j * ldx + i] - geo->c[j]) / Reff;
        rho2 = rho2 + v * v;
      }
      tt[e] = (T)((2.0 * rho2 - u0 - u1) / (u1 - u0));
    }
  }
  for (int row = 0; row < S; ++row) {
    const int L = q_len[row];
    const T* cf = coef + q_off[row];
    T b1[PPT], b2[PPT], val[PPT];
#pragma unroll
    for (int e = 0; e < PPT; ++e) { b1[e] = 0; b2[e] = 0; }
    for (int a = L - 1; a >= 1; --a) {
      const T c = cf[a];
#pragma unroll
      for (int e = 0; e < PPT; ++e) {
        const T b0 = 2 * tt[e] * b1[e] - b2[e] + c;
        b2[e] = b1[e];
        b1[e] = b0;
      }
    }
#pragma unroll
    for (int e = 0; e < PPT; ++e) val[e] = i0 + e < n ? scale * (tt[e] * b1[e] - b2[e] + cf[0]) : (T)0;
    store_row<T, PPT>(out + (int64_t)row * ld_out + i0, val);
  }
}

hipError_t launch_radial(const void* x_soa, int dtype, int64_t ldx, int64_t n, int d, const GeoDev* geo,
                         double u0, double u1, const int32_t* q_len, const int32_t* q_off, const void* coef,
                         int S, double scale, int prec, void* out, int64_t ld_out, hipStream_t s) {
  if (S <= 0 || n <= 0) return hipSuccess;
  if (ld_out < row_end(n)) return hipErrorInvalidValue;
#define HDF_RAD(TIN, T)                                                                                      \
  do {                                                                                                       \
    constexpr int PPT = 16 / sizeof(T);                                                                      \
    const unsigned nb = (unsigned)((row_end(n) + 256 * PPT - 1) / (256 * PPT));                             \
    k_radial<TIN, T, PPT><<<nb, 256, 0, s>>>((const TIN*)x_soa, ldx, n, d, geo, u0, u1, q_len, q_off,       \
                                             (const T*)coef, S, (T)scale, (T*)out, ld_out);                  \
  } while (0)
  if (prec == 1 && dtype == 0) HDF_RAD(float, float);
  else if (prec == 0 && dtype == 1) HDF_RAD(double, double);
  else if (prec == 0 && dtype == 0) HDF_RAD(float, double);
  else return hipErrorInvalidValue;
#undef HDF_RAD
  return hipGetLastError();
}

// dX[i][j] = (1/R) [ sum_c w_ic KS[i][j 2m + c] + v_ic KS[i][j 2m + m + c]
//                    + 2 xt_ij (sum_c w_ic K2[i][c] + v_ic K2[i][m + c]) ]
// KS: n x ldks (the shifted-factor products, 2m columns per direction; null: zeros), K2: n x ldk2.
template <typename Tin, typename T, typename TIO>
__global__ void __launch_bounds__(256) k_adj_combine(const Tin* __restrict__ x_soa, int64_t ldx, int64_t n, int d,
                                                      const GeoDev* __restrict__ geo, const T* __restrict__ KS,
                                                      int64_t ldks, const T* __restrict__ K2, int64_t ldk2,
                                                      const TIO* __restrict__ Wm, const TIO* __restrict__ Vm,
                                                      int64_t ld, int m, TIO* __restrict__ dX, int64_t lddx) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double Reff = geo->Reff;
  double s2 = 0.0;
  for (int c = 0; c < m; ++c)
    s2 += (double)Wm[i * ld + c] * (double)K2[i * ldk2 + c] + (double)Vm[i * ld + c] * (double)K2[i * ldk2 + m + c];
  for (int j = 0; j < d; ++j) {
    double sj = 0.0;
    const T* ks = KS ? KS + i * ldks + (int64_t)j * 2 * m : nullptr;
    for (int c = 0; c < m; ++c)
      sj += (double)Wm[i * ld + c] * (ks ? (double)ks[c] : 0.0) + (double)Vm[i * ld + c] * (ks ? (double)ks[m + c] : 0.0);
    const double xt = ((double)x_soa[(int64_t)j * ldx + i] - geo->c[j]) / Reff;
    dX[i * lddx + j] = (TIO)((sj + 2.0 * xt * s2) / Reff);
  }
}

hipError_t launch_adj_combine(const void* x_soa, int dtype, int64_t ldx, int64_t n, int d, const GeoDev* geo,
                              const void* KS, int64_t ldks, const void* K2, int64_t ldk2, const void* Wm,
                              const void* Vm, int64_t ld, int m, void* dX, int64_t lddx, int prec, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const unsigned nb = (unsigned)((n + 255) / 256);
#define HDF_COMB(TIN, T)                                                                                     \
  k_adj_combine<TIN, T, TIN><<<nb, 256, 0, s>>>((const TIN*)x_soa, ldx, n, d, geo, (const T*)KS, ldks,      \
                                                (const T*)K2, ldk2, (const TIN*)Wm, (const TIN*)Vm, ld, m,   \
                                                (TIN*)dX, lddx)
  if (prec == 1 && dtype == 0) HDF_COMB(float, float);
  else if (prec == 0 && dtype == 1) HDF_COMB(double, double);
  else if (prec == 0 && dtype == 0) HDF_COMB(float, double);
  else return hipErrorInvalidValue;
#undef HDF_COMB
  return hipGetLastError();
}

// Pass 1, tile-major.  Per degree k, W_k = Phi_k (Q_k o V): every wave item
// owns one 16-row tile of Phi_k and up to eight accumulator tiles (radial
// function l, column tile ct), so one pair of 16-byte loads of the tile's
// values per lane and 32-point chunk feeds 8 * nl * nct MFMAs.  MFMA K-step t
// of a chunk takes the four points p + 8 g + t (lane group g) with
//   A[r][g] = phi_{row0 + r}(p + 8 g + t) q_l(p + 8 g + t),
//   B[g][c] = V[p + 8 g + t][16 ct + c],
// A formed from the tile's values and the staged radial rows, B from V^T in LDS.  A rank-row item
// (MvtRankRow) takes row r's harmonic and radial row from its own table entry.  The tile's values are
// prefetched PF chunks ahead into registers; the staged operands (V^T and the
// radial rows) are staged for two chunks at a time into double-buffered LDS,
// with one barrier per such unit.  Every load is unconditional and in
// bounds: chunk and unit starts are clamped to the split's last chunk and
// unit, Phi and Q rows are padded by at least 63 points past n (zeros), V rows
// are clamped to n - 1 and the values of points past the split multiplied by
// zero.
// More than 64 columns run in slabs of 64 (blockIdx.y) into their columns of rows of mo entries: the
// staged V^T of 64 columns is what LDS and the accumulators take, and a slab is bound by the matrix
// cores, so reading the tile again costs nothing.  Products of more than 64 columns with the
// per-column-tile kernel before and now: 1e6 points x 168 18.9 and 12.3 ms, 100,003 x 128 binary64 5.1 and
// 3.5, 44,599 x 80 0.31 and 0.18, 9,973 x 100 0.21 and 0.09.
// Prefetch depth (chunks of the tile in flight) and occupancy per type and column tiles, chosen so
// that the loops hold their registers: binary32 at four wavefronts per SIMD (<= 128 registers, two
// workgroups on a CU), with one column tile 4 chunks deep, otherwise 2; binary64 two with one column
// tile (117 registers all the same), three with more.  Binary32 with four column tiles spills one
// register around the loop: at three wavefronts (132 registers, one workgroup on a CU) 64 columns on 1e6
// points took 2.31 ms instead of 2.04.  Binary64 with more column tiles spills inside the loop at four: the
// product of 64 columns took 7.1 ms instead of 4.5, of 32 columns 1.71 instead of 1.46.
// Without the occupancy hint the scheduler hoists the operands of all radial functions and
// overflows the registers.
template <typename T, int NCT> struct MvtPF { static constexpr int value = sizeof(T) == 4 && NCT == 1 ? 4 : 2; };
template <typename T, int NCT> struct MvtWaves {
  static constexpr int value = sizeof(T) == 4 ? 4 : (NCT == 1 ? 2 : 3);
};
// radial functions per wave item (accumulator tiles per wavefront: NL * NCT); binary32 with two
// column tiles keeps three, the registers of four spill
template <typename T, int NCT> struct MvtNL {
  static constexpr int value = sizeof(T) == 4 ? (NCT == 2 ? 3 : 8 / NCT) : 4 / NCT;
};
constexpr int kMvtCH = 32;                 // points per chunk (MFMA K-steps of one tile load)
constexpr int kMvtSP = 2;                  // chunks per staged unit (one barrier per unit)
constexpr int kMvtSpan = kMvtSP * kMvtCH;  // points per staged unit
constexpr int kMvtThreads = 64 * kMvtWavesPerGroup;
constexpr int kMvtVS = kMvtSpan + 4;       // padded staged row (LDS bank spread)


template <typename T, typename TV, int NCT>
__device__ __forceinline__ void mvt_tile(int b, const T* __restrict__ phi, int64_t ld_phi,
                                         const T* __restrict__ q, int64_t ld_q, const MvtWave* __restrict__ waves,
                                         const MvtRankRow* __restrict__ rrows, const MvtGroup* __restrict__ groups,
                                         int n_groups, int n_splits, int64_t split_len, const TV* __restrict__ V,
                                         int64_t ldv, int64_t n, int m, int m16, int mo, int64_t rank,
                                         double* __restrict__ part) {
  typedef typename Mfma<T>::V Acc;
  constexpr int PF = MvtPF<T, NCT>::value;
  static_assert(PF % 2 == 0, "the LDS buffer of a chunk is its slot's parity");
  constexpr int NL = MvtNL<T, NCT>::value;
  constexpr int CH = kMvtCH, VS = kMvtVS, SP = kMvtSP, SPAN = kMvtSpan;
  static_assert(PF % SP == 0, "whole staged units in flight");
  constexpr int PS = PF / SP;                       // staged units in flight
  extern __shared__ unsigned char smem_raw[];
  T* lds = reinterpret_cast<T*>(smem_raw);
  // block b runs group gi over split sp with b = 8 (G (sp / 8) + gi) + sp % 8: the workgroups of
  // all groups over one range of points land on one XCD (dispatch is round robin over the eight),
  // close together in time, so V and the radial rows of the range are fetched into its L2 once
  const int rest = b >> 3;
  const int gi = rest % n_groups;
  const int split = ((rest / n_groups) << 3) + (b & 7);
  if (split >= n_splits) return;                    // whole workgroup, before any barrier
  const MvtGroup gd = groups[gi];
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool active = wave < gd.nw;                 // uniform
  const MvtWave wi = waves[gd.w0 + (active ? wave : 0)];
  const int64_t p_begin = (int64_t)split * split_len;
  const int64_t p_end = (p_begin + split_len < n) ? p_begin + split_len : n;
  const int64_t p_last = p_begin + (p_end - 1 - p_begin) / CH * CH;   // start of the split's last chunk
  const int64_t u_last = p_begin + (p_end - 1 - p_begin) / SPAN * SPAN;   // ... and of its last unit
  const int half = (m16 + kMvtMaxNq + 1) * VS;      // one buffer: V^T (m16 rows), radial rows, a pad row
  // this lane's Phi row and first staged radial row (rows past the tile repeat its first row; their
  // outputs are not written); a rank-row item gives each lane its own pair
  const bool rank_item = wi.qrow < 0;               // uniform
  int hrow = wi.row0 + (li < wi.nr ? li : 0), qlane = wi.qrow - gd.q_lo;
  if (rank_item) {
    const MvtRankRow rr = rrows[wi.row0 + (li < wi.nr ? li : 0)];
    hrow = rr.hrow;
    qlane = rr.qrow - gd.q_lo;
  }
  const T* prow = phi + (int64_t)hrow * ld_phi + 8 * g;

  auto load_tile = [&](int64_t p, T (&a)[8]) {
    const int64_t pc = p < p_last ? p : p_last;
    const T* r = prow + pc;
    if constexpr (sizeof(T) == 4) {
      const floatx4 v0 = *reinterpret_cast<const floatx4*>(r);
      const floatx4 v1 = *reinterpret_cast<const floatx4*>(r + 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) { a[e] = v0[e]; a[4 + e] = v1[e]; }
    } else {
#pragma unroll
      for (int h = 0; h < 4; ++h) {
        const doublex2 w = *reinterpret_cast<const doublex2*>(r + 2 * h);
        a[2 * h] = w[0];
        a[2 * h + 1] = w[1];
      }
    }
  };
  // staging of a unit (SPAN = 64 points, two chunks) by all threads (TPB of them): V entries
  // e = tid + TPB j < 64 m16 (point e / m16, column e % m16) and the group's radial entries, SQ
  // consecutive points of one row per thread (row SQ tid / 64; rows past nq repeat the last one and
  // are never read).  The loads are unconditional and in bounds and keep the raw values; the masks
  // (points past the split, columns past m) and the choice of slot are applied when the values are
  // written to LDS, so the compiler's load-counter waits stay exact (a select right after a load,
  // or a branch around it, makes it wait for every load in flight).
  constexpr int TPB = kMvtThreads;
  constexpr int SV = (SPAN * 16 * NCT + TPB - 1) / TPB, SQ = SPAN * kMvtMaxNq / TPB;
  static_assert(SQ == 2 || SQ == 4, "radial staging: two or four consecutive points per thread");
  typedef T T2 __attribute__((ext_vector_type(2)));
  const int sv_n = SPAN * m16;                       // staged V entries per unit
  // e / m16 for the staged entries e < 4096 as (e * inv16) >> 20: exact for m16 <= 64 (the error
  // of the rounded-up reciprocal stays below 2^-8 < 1 / m16)
  const uint32_t inv16 = ((1u << 20) + (uint32_t)m16 - 1) / (uint32_t)m16;
  static_assert(TPB * SV <= 4096, "staged entry index range of the reciprocal division");
  // staged values are loaded with the same look-ahead as the tile (PF chunks = PS units, rotating
  // register slots): the load counter completes in issue order, so values loaded after the tile
  // prefetch could only be waited for together with it
  TV sv[PS][SV];
  T sq[PS][SQ];
  auto stage_load = [&](int64_t p0, TV (&sv)[SV], T (&sq)[SQ]) {
    const int64_t p = p0 < u_last ? p0 : u_last;
#pragma unroll
    for (int j = 0; j < SV; ++j) {
      const int e = tid + TPB * j;
      const int pp = (int)(((uint32_t)e * inv16) >> 20), c = e - pp * m16;
      const int64_t pt = p + pp;
      const int64_t ptc = pt < n ? pt : n - 1;
      sv[j] = V[ptc * ldv + (c < m ? c : 0)];
    }
    const int e = SQ * tid;
    const int r = e / SPAN, pq = e % SPAN;
    const int rc = r < gd.nq ? r : gd.nq - 1;
    const T* src = q + (int64_t)(gd.q_lo + rc) * ld_q + p + pq;
#pragma unroll
    for (int h = 0; h < SQ / 2; ++h) {
      const T2 w = *reinterpret_cast<const T2*>(src + 2 * h);
      sq[2 * h] = w[0];
      sq[2 * h + 1] = w[1];
    }
  };
  // values of the unit starting at p into buf; entries past the staged area go to the pad row
  auto stage_store = [&](T* buf, int64_t p, const TV (&sv)[SV], const T (&sq)[SQ]) {
#pragma unroll
    for (int j = 0; j < SV; ++j) {
      const int e = tid + TPB * j;
      const int pp = (int)(((uint32_t)e * inv16) >> 20), c = e - pp * m16;
      const bool ok = p + pp < p_end && c < m;
      const int at = e < sv_n ? c * VS + pp : (m16 + kMvtMaxNq) * VS + (tid & 63);
      buf[at] = ok ? (T)sv[j] : (T)0;
    }
    const int e = SQ * tid;
    T* dst = buf + m16 * VS + (e / SPAN) * VS + e % SPAN;
#pragma unroll
    for (int h = 0; h < SQ / 2; ++h) {
      T2 w;
      w[0] = sq[2 * h];
      w[1] = sq[2 * h + 1];
      *reinterpret_cast<T2*>(dst + 2 * h) = w;
    }
  };
  auto lds8 = [&](const T* p, T (&v)[8]) {
    if constexpr (sizeof(T) == 4) {
      const floatx4 a = *reinterpret_cast<const floatx4*>(p), b = *reinterpret_cast<const floatx4*>(p + 4);
#pragma unroll
      for (int t = 0; t < 4; ++t) { v[t] = a[t]; v[4 + t] = b[t]; }
    } else {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const double2 a = *reinterpret_cast<const double2*>(p + 2 * t);
        v[2 * t] = a[0];
        v[2 * t + 1] = a[1];
      }
    }
  };

  Acc acc[NL][NCT];
#pragma unroll
  for (int j = 0; j < NL; ++j)
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) acc[j][ct] = Acc{0, 0, 0, 0};
  // tile slot j holds chunk c = j (mod PF); staged slot u holds unit U = u (mod PS).  The chunk loop
  // runs in whole groups of PF chunks; chunks past the split load clamped, in-bounds data and meet
  // zero V values, so they add nothing.
  T a[PF][8];
#pragma unroll
  for (int j = 0; j < PF; ++j) load_tile(p_begin + j * CH, a[j]);
#pragma unroll
  for (int u = 0; u < PS; ++u) stage_load(p_begin + u * SPAN, sv[u], sq[u]);
  stage_store(lds, p_begin, sv[0], sq[0]);
  stage_load(p_begin + PS * SPAN, sv[0], sq[0]);    // slot 0 next holds unit PS
  __syncthreads();
  const int64_t n_chunks = (p_end - p_begin + CH - 1) / CH;
  const int64_t n_rounds = (n_chunks + PF - 1) / PF;
  for (int64_t it = 0; it < n_rounds; ++it) {
#pragma unroll
    for (int j = 0; j < PF; ++j) {
      const int64_t pc = p_begin + (it * PF + j) * CH;
      const int buf = (int)((it * PS + j / SP) & 1);  // the unit's LDS buffer: its parity
      const T* cur = lds + buf * half + (j % SP) * CH;
      if (active) {                                 // uniform
        // radial function outermost: the A operands (tile values times the radial row) are formed
        // once and serve every column tile
#pragma unroll
        for (int l = 0; l < NL; ++l) {
          if (l < wi.nl) {                          // uniform
            T av[8];
            lds8(cur + m16 * VS + (qlane + l) * VS + 8 * g, av);
#pragma unroll
            for (int t = 0; t < 8; ++t) av[t] *= a[j][t];
#pragma unroll
            for (int ct = 0; ct < NCT; ++ct) {
              if (ct < wi.nct) {                    // uniform
                T v[8];
                lds8(cur + (16 * (wi.ct0 + ct) + li) * VS + 8 * g, v);
#pragma unroll
                for (int t = 0; t < 8; ++t) acc[l][ct] = Mfma<T>::run(av[t], v[t], acc[l][ct]);
              }
              // column tiles one after the other: hoisting the operands of all of them overflows
              // the registers of the binary64 shapes and of binary32 with two column tiles
              if constexpr (sizeof(T) == 8 || NCT == 2) __builtin_amdgcn_sched_barrier(0);
            }
          }
        }
      }
      load_tile(pc + PF * CH, a[j]);
      if (j % SP == SP - 1) {
        // end of unit U: unit U + 1 (slot (U + 1) mod PS) goes to the other buffer, and the slot
        // is refilled with unit U + 1 + PS
        const int slot = (j / SP + 1) % PS;
        stage_store(lds + (buf ^ 1) * half, pc + CH, sv[slot], sq[slot]);
        stage_load(pc + CH + PS * SPAN, sv[slot], sq[slot]);
        __syncthreads();
      }
    }
  }
  if (!active) return;
  double* out = part + (int64_t)split * rank * mo;
  if (rank_item) {
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) {
      if (ct < wi.nct) {
        const int c = 16 * (wi.ct0 + ct) + li;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int r = Mfma<T>::row(g, e);
          if (r < wi.nr) out[(int64_t)rrows[wi.row0 + r].out * mo + c] = (double)acc[0][ct][e];
        }
      }
    }
    return;
  }
#pragma unroll
  for (int l = 0; l < NL; ++l) {
    if (l < wi.nl) {
#pragma unroll
      for (int ct = 0; ct < NCT; ++ct) {
        if (ct < wi.nct) {
          const int c = 16 * (wi.ct0 + ct) + li;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int h = Mfma<T>::row(g, e);
            if (h < wi.nr) out[(int64_t)(wi.out0 + h * wi.s + l) * mo + c] = (double)acc[l][ct][e];
          }
        }
      }
    }
  }
}

template <typename T, typename TV, int NCT>
__global__ void __launch_bounds__(kMvtThreads) __attribute__((amdgpu_waves_per_eu(MvtWaves<T, NCT>::value, 8)))
k_mv_t_tile(const T* __restrict__ phi, int64_t ld_phi, const T* __restrict__ q, int64_t ld_q,
            const MvtWave* __restrict__ waves, const MvtRankRow* __restrict__ rrows,
            const MvtGroup* __restrict__ groups, int n_groups, int n_splits, int64_t split_len,
            const TV* __restrict__ V, int64_t ldv, int64_t n, int m, int m16, int mo, int64_t rank,
            double* __restrict__ part) {
  const int c0 = blockIdx.y * m16;                  // the slab's first column
  mvt_tile<T, TV, NCT>(blockIdx.x, phi, ld_phi, q, ld_q, waves, rrows, groups, n_groups, n_splits, split_len, V + c0, ldv,
                       n, m - c0, m16, mo, rank, part + c0);
}

int matvec_tile_nl(int prec, int nct) {
  if (prec == 1) return nct == 1 ? MvtNL<float, 1>::value : (nct == 2 ? MvtNL<float, 2>::value : MvtNL<float, 4>::value);
  return nct == 1 ? MvtNL<double, 1>::value : (nct == 2 ? MvtNL<double, 2>::value : MvtNL<double, 4>::value);
}

size_t matvec_tile_lds_bytes(int m16, int prec) {
  return 2 * (size_t)(m16 + kMvtMaxNq + 1) * kMvtVS * (prec == 1 ? 4 : 8);
}

hipError_t launch_matvec_t_tile(const void* phi, int64_t ld_phi, const void* q, int64_t ld_q,
                                const MvtWave* waves, const MvtRankRow* rank_rows, const MvtGroup* groups,
                                int n_groups, int n_splits,
                                int64_t split_len, const void* V, int64_t ldv, int64_t n, int m, int m16,
                                int n_slabs, int mo, int64_t rank, double* partials, int prec, int io, hipStream_t s) {
  if (m16 < 16 || m16 > 64 || m16 % 16 || n_slabs < 1 || mo < n_slabs * m16 || m <= (n_slabs - 1) * m16 ||
      n_groups < 1 || n_splits < 1 || split_len % kMvtCH)
    return hipErrorInvalidValue;
  if ((int64_t)(n_splits - 1) * split_len >= n || (int64_t)n_splits * split_len < n) return hipErrorInvalidValue;
  const int cpl = m16 / 16;
  const size_t lds = matvec_tile_lds_bytes(m16, prec);
  const unsigned n_blocks = (unsigned)(((n_splits + 7) / 8) * 8 * n_groups);
#define HDF_MVTT(T, TV, NC)                                                                                   \
  k_mv_t_tile<T, TV, NC><<<dim3(n_blocks, n_slabs), kMvtThreads, lds, s>>>((const T*)phi, ld_phi, (const T*)q, ld_q, waves,          \
                                                    rank_rows, groups,                                        \
                                                    n_groups, n_splits, split_len, (const TV*)V, ldv, n, m,   \
                                                    m16, mo, rank, partials)
#define HDF_MVTT_NCT(T, TV)                                                                                   \
  do {                                                                                                        \
    if (cpl == 1) HDF_MVTT(T, TV, 1);                                                                         \
    else if (cpl == 2) HDF_MVTT(T, TV, 2);                                                                    \
    else HDF_MVTT(T, TV, 4);                                                                                  \
  } while (0)
  if (prec == 1 && io == 0) HDF_MVTT_NCT(float, float);
  else if (prec == 0 && io == 1) HDF_MVTT_NCT(double, double);
  else if (prec == 0 && io == 0) HDF_MVTT_NCT(double, float);
  else return hipErrorInvalidValue;
#undef HDF_MVTT_NCT
#undef HDF_MVTT
  return hipGetLastError();
}

// Fixed-order reduction over the pass-1 splits, one wavefront-wide group of 64 entries per workgroup:
// wavefront w takes the splits w, w + 4, ... with eight running sums (loads in flight), and the four
// sums are combined in a fixed order.  The entries run over the blocks of pass 2 (16 harmonics x one
// radial function, `src` their rank rows, -1 past a degree's harmonics) and the m16 columns; each sum
// goes to W (rank rows), to the scaled copy Wd = D W (rank rows) and to Wb, the scaled copy in pass
// 2's order: block, 16-column tile, then (lane 16 g + c, K-step kb) for harmonic 4 kb + g, zeros past
// the degree's harmonics.  Any of the three may be null.
template <typename T>
__device__ __forceinline__ void mv_reduce(int bx, const double* __restrict__ part, int n_splits, int64_t stride,
                                          int64_t total, int m16, const int32_t* __restrict__ src,
                                          const double* __restrict__ lam_row, double* __restrict__ W,
                                          T* __restrict__ Wd, T* __restrict__ Wb) {
  __shared__ double red[4][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t e = (int64_t)bx * 64 + lane;
  const int64_t row = e < total ? e / m16 : 0;
  const int c = (int)(e < total ? e - row * m16 : 0);
  const int sr = e < total ? src[row] : -1;
  const double* p = part + (int64_t)(sr < 0 ? 0 : sr) * m16 + c;
  double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  int sp = w;
  for (; sp + 28 < n_splits; sp += 32)
#pragma unroll
    for (int u = 0; u < 8; ++u) acc[u] += p[(int64_t)(sp + 4 * u) * stride];
  for (; sp < n_splits; sp += 4) acc[0] += p[(int64_t)sp * stride];
  red[w][lane] = ((acc[0] + acc[1]) + (acc[2] + acc[3])) + ((acc[4] + acc[5]) + (acc[6] + acc[7]));
  __syncthreads();
  if (w != 0 || e >= total) return;
  const double v = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
  const T sc = sr < 0 ? (T)0 : (T)(lam_row[sr < 0 ? 0 : sr] * v);
  if (sr >= 0 && W) W[(int64_t)sr * m16 + c] = v;
  if (sr >= 0 && Wd) Wd[(int64_t)sr * m16 + c] = sc;
  if (Wb) {
    const int hh = (int)(row & 15), kb = hh >> 2, g = hh & 3;
    Wb[((row >> 4) * (m16 >> 4) + (c >> 4)) * 256 + (g * 16 + (c & 15)) * 4 + kb] = sc;
  }
}

template <typename T>
__global__ void __launch_bounds__(256) k_mv_reduce(const double* __restrict__ part, int n_splits, int64_t stride,
                                                    int64_t total, int m16, const int32_t* __restrict__ src,
                                                    const double* __restrict__ lam_row, double* __restrict__ W,
                                                    T* __restrict__ Wd, T* __restrict__ Wb) {
  mv_reduce(blockIdx.x, part, n_splits, stride, total, m16, src, lam_row, W, Wd, Wb);
}

// Pass 2, KV = U (D W).  One wavefront owns 64 points and NCT 16-column tiles of the right-hand sides.
// The reduction runs over the rank columns (k, h, l) directly: the MFMA A operand is
// U[i, (k,h,l)] = phi_h(i) q_{k,l}(i), formed in registers from the harmonic rows and the points'
// radial values, and B is row (k,h,l) of D W.  The accumulators (one per point tile and column tile)
// are the output itself.  MFMA row i of point tile u is point p0 + 4 i + u, so each lane reads 4
// consecutive points of a harmonic (or radial) row with 16-byte loads, and the four values of D W that
// a lane needs for a block (16 harmonics, one radial function: four K-steps) are one 16-byte
// (32-byte) load of Wb (k_mv_reduce).
// What bounds it: memory with one column tile, the matrix cores with four.  So the harmonic rows and
// the operands U are formed once for up to four column tiles, and the number of radial functions is a
// template parameter: a batch of 16 harmonics is then one block of straight code, in which the waits
// for the operands of radial function l + 1 and for the next batch's rows are counted, not taken for
// every load in flight as around a loop over l.  Rows past a degree's harmonics are those of the next
// degree (the last row past the last) and meet zero rows of Wb; points past n are read from the rows' padding and not written.
// With z_blocks > 0 (few points) blockIdx.z takes the blocks [z z_blocks, (z + 1) z_blocks) only,
// whatever degree and radial function they are, and writes its share of KV to part[z][n][m];
// k_mv_n_sum adds the shares in z order.
// 64 columns: binary32, 1e6 points, rank 1413 3.06 -> 1.88 ms (96 TFLOP/s);
// binary64, 5e5 points, rank 1463 4.43 -> 2.08 ms (45 TFLOP/s; two column tiles per wavefront 2.22).
// 16 columns: binary64, 250,007 points 0.73 -> 0.52 ms; binary32, 1e6 points 0.79 -> 0.78 ms (memory).
// Wavefronts per SIMD that the registers are held to (accumulators: 16 NCT registers in binary32,
// 32 NCT in binary64):
template <typename T, int NCT> struct MvnWaves {
  static constexpr int value = sizeof(T) == 4 ? (NCT == 1 ? 4 : (NCT == 2 ? 3 : 2)) : (NCT == 1 ? 2 : 1);
};
constexpr int kMvnKB = 4;                          // K-steps per block: 16 harmonics

// four consecutive points of a padded row (in bounds up to 63 points past n)
template <typename T>
__device__ __forceinline__ void mvn_load4(const T* __restrict__ p, T (&o)[4]) {
  if constexpr (sizeof(T) == 4) {
    const floatx4 w = *reinterpret_cast<const floatx4*>(p);
#pragma unroll
    for (int u = 0; u < 4; ++u) o[u] = w[u];
  } else {
    const doublex2 w0 = *reinterpret_cast<const doublex2*>(p);
    const doublex2 w1 = *reinterpret_cast<const doublex2*>(p + 2);
    o[0] = w0[0]; o[1] = w0[1]; o[2] = w1[0]; o[3] = w1[1];
  }
}

template <typename T, int NCT>
struct MvnPass {
  typedef typename Mfma<T>::V Acc;
  // wavefront-uniform bases and this lane's offsets (values): the loads take their base from scalar registers
  const T* phi;                                    // at the first of the wavefront's points
  const T* q;
  const T* wb;                                     // first column tile of the group
  int64_t ld_phi, ld_q, wb_stride;                 // wb_stride: values per block
  int ct_off[NCT];                                 // column tile offsets in a block (uniform)
  int last_row;                                    // last harmonic row of phi
  int g;
  uint32_t pt_off, wb_off;                         // 4 li, lane kMvnKB
  Acc acc[NCT][4];

  __device__ __forceinline__ void rows(const DegDev& dg, int b, T (&v)[kMvnKB][4]) const {
#pragma unroll
    for (int kb = 0; kb < kMvnKB; ++kb) {
      const int row = dg.hoff + 16 * b + 4 * kb + g;
      mvn_load4(phi + (int64_t)(row < last_row ? row : last_row) * ld_phi + pt_off, v[kb]);
    }
  }
  __device__ __forceinline__ void operands(int qrow, int64_t block, T (&ql)[4], T (&bw)[NCT][kMvnKB]) const {
    const T* qb = q + (int64_t)qrow * ld_q;
    const T* wbb = wb + block * wb_stride;
    mvn_load4(qb + pt_off, ql);
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) mvn_load4(wbb + ct_off[ct] + wb_off, bw[ct]);
  }
  __device__ __forceinline__ void multiply(const T (&v)[kMvnKB][4], const T (&ql)[4], const T (&bw)[NCT][kMvnKB]) {
#pragma unroll
    for (int kb = 0; kb < kMvnKB; ++kb) {
      T av[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) av[u] = v[kb][u] * ql[u];
#pragma unroll
      for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
        for (int u = 0; u < 4; ++u) acc[ct][u] = Mfma<T>::run(av[u], bw[ct][kb], acc[ct][u]);
    }
  }
  // radial functions [l0, l0 + SN) of all batches of a degree
  template <int SN>
  __device__ __forceinline__ void degree(const DegDev& dg, int l0) {
    const int nb = (dg.nh + 15) >> 4;
    T vn[kMvnKB][4], ql[2][4], bw[2][NCT][kMvnKB];
    // the indices are carried from load to load through readfirstlane, so that the compiler forms each
    // address when it is needed instead of holding those of every radial function in registers
    int qr = dg.qoff + l0, blk = dg.boff + l0;
    operands(qr, blk, ql[0], bw[0]);
    rows(dg, 0, vn);
    for (int b = 0; b < nb; ++b) {
      const int bn = b + 1 < nb ? b + 1 : b;
      T v[kMvnKB][4];
#pragma unroll
      for (int kb = 0; kb < kMvnKB; ++kb)
#pragma unroll
        for (int u = 0; u < 4; ++u) v[kb][u] = vn[kb][u];
#pragma unroll
      for (int l = 0; l < SN; ++l) {
        // the operands of the next radial function, or those of the next batch's first
        qr = __builtin_amdgcn_readfirstlane(l + 1 < SN ? qr + 1 : qr - (SN - 1));
        blk = __builtin_amdgcn_readfirstlane(l + 1 < SN ? blk + 1 : blk - (SN - 1) + (bn - b) * dg.s);
        operands(qr, blk, ql[(l + 1) & 1], bw[(l + 1) & 1]);
        if (l == 0) rows(dg, bn, vn);
        __builtin_amdgcn_sched_barrier(0);
        multiply(v, ql[l & 1], bw[l & 1]);
      }
      if constexpr (SN & 1) {
#pragma unroll
        for (int u = 0; u < 4; ++u) ql[0][u] = ql[1][u];
#pragma unroll
        for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
          for (int kb = 0; kb < kMvnKB; ++kb) bw[0][ct][kb] = bw[1][ct][kb];
      }
    }
  }
};

template <typename T, typename TO, int NCT, bool SPLIT>
__device__ __forceinline__ void mv_n(unsigned bx, int bz, const T* __restrict__ phi, int64_t ld_phi,
                                     const T* __restrict__ q, int64_t ld_q, const DegDev* __restrict__ degs, int n_deg,
                                     const T* __restrict__ Wb, int m16, TO* __restrict__ KV, int64_t ldkv, int64_t n,
                                     int m, int z_blocks, int n_blocks, T* __restrict__ part) {
  const int lane = threadIdx.x, li = lane & 15, g = lane >> 4;
  // block b takes column group cg of point block pb, b = 8 (n_cg (pb / 8) + cg) + pb % 8: the column
  // groups of a point block run on one XCD (dispatch is round robin over the eight), close in time,
  // and share the harmonic rows in its L2
  const int cpl = m16 >> 4, n_cg = (cpl + NCT - 1) / NCT;
  const int rest = (int)(bx >> 3), cg = rest % n_cg;
  const int64_t p0 = ((int64_t)(rest / n_cg) * 8 + (bx & 7)) * 64;
  if (p0 >= n) return;
  const int ct0 = cg * NCT, nct = cpl - ct0 < NCT ? cpl - ct0 : NCT;   // column tiles of this group
  MvnPass<T, NCT> ps;
  ps.phi = phi + p0;
  ps.q = q + p0;
  ps.wb = Wb + (int64_t)ct0 * 256;
  ps.pt_off = 4 * li;
  ps.wb_off = lane * kMvnKB;
  ps.last_row = degs[n_deg - 1].hoff + degs[n_deg - 1].nh - 1;
  ps.ld_phi = ld_phi;
  ps.ld_q = ld_q;
  ps.wb_stride = (int64_t)cpl * 256;
  ps.g = g;
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct) {
    // a column tile past the last repeats the group's first (never written)
    ps.ct_off[ct] = ct < nct ? ct * 256 : 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) ps.acc[ct][u] = typename Mfma<T>::V{0, 0, 0, 0};
  }
  if constexpr (!SPLIT) {
    for (int di = 0; di < n_deg; ++di) {
      const DegDev dg = degs[di];
      for (int l0 = 0; l0 < dg.s; l0 += 8) {
        switch (dg.s - l0) {                       // uniform
          case 1: ps.template degree<1>(dg, l0); break;
          case 2: ps.template degree<2>(dg, l0); break;
          case 3: ps.template degree<3>(dg, l0); break;
          case 4: ps.template degree<4>(dg, l0); break;
          case 5: ps.template degree<5>(dg, l0); break;
          case 6: ps.template degree<6>(dg, l0); break;
          case 7: ps.template degree<7>(dg, l0); break;
          default: ps.template degree<8>(dg, l0); break;
        }
      }
    }
  } else {
    // block after block, the next one's rows and operands in flight
    int blk = bz * z_blocks;
    const int hi = blk + z_blocks < n_blocks ? blk + z_blocks : n_blocks;
    int di = 0;
    while (di + 1 < n_deg && degs[di + 1].boff <= blk) ++di;
    DegDev dg = degs[di];
    int b = (blk - dg.boff) / dg.s, l = (blk - dg.boff) % dg.s;
    T vn[kMvnKB][4], qn[4], wn[NCT][kMvnKB];
    ps.operands(dg.qoff + l, blk, qn, wn);
    ps.rows(dg, b, vn);
    for (; blk < hi; ++blk) {
      T v[kMvnKB][4], ql[4], bw[NCT][kMvnKB];
#pragma unroll
      for (int kb = 0; kb < kMvnKB; ++kb)
#pragma unroll
        for (int u = 0; u < 4; ++u) v[kb][u] = vn[kb][u];
#pragma unroll
      for (int u = 0; u < 4; ++u) ql[u] = qn[u];
#pragma unroll
      for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
        for (int kb = 0; kb < kMvnKB; ++kb) bw[ct][kb] = wn[ct][kb];
      if (++l == dg.s) {
        l = 0;
        ++b;
      }
      if (16 * b >= dg.nh) {                       // past the degree: the next one's first block
        b = 0;
        if (di + 1 < n_deg) dg = degs[++di];
      }
      ps.operands(dg.qoff + l, blk + 1 < hi ? blk + 1 : blk, qn, wn);
      ps.rows(dg, b, vn);
      __builtin_amdgcn_sched_barrier(0);
      ps.multiply(v, ql, bw);
    }
  }
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct) {
    const int c = 16 * (ct0 + ct) + li;
    if (ct < nct && c < m) {
      T* dpart = SPLIT ? part + (int64_t)bz * n * m : nullptr;
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int64_t pt = p0 + 4 * Mfma<T>::row(g, e) + u;
          if (pt < n) {
            if constexpr (SPLIT) dpart[pt * m + c] = ps.acc[ct][u][e];
            else KV[pt * ldkv + c] = (TO)ps.acc[ct][u][e];
          }
        }
    }
  }
}

template <typename T, typename TO, int NCT, bool SPLIT>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(MvnWaves<T, NCT>::value, 8)))
k_mv_n(const T* __restrict__ phi, int64_t ld_phi, const T* __restrict__ q, int64_t ld_q,
       const DegDev* __restrict__ degs, int n_deg, const T* __restrict__ Wb, int m16, TO* __restrict__ KV,
       int64_t ldkv, int64_t n, int m, int z_blocks, int n_blocks, T* __restrict__ part) {
  mv_n<T, TO, NCT, SPLIT>(blockIdx.x, blockIdx.z, phi, ld_phi, q, ld_q, degs, n_deg, Wb, m16, KV, ldkv, n, m, z_blocks,
                          n_blocks, part);
}

// Sum of pass 2's shares in a fixed order: a workgroup owns 64 entries, wavefront w takes the shares
// w, w + 4, ... with four running sums (one thread per entry over 128 shares of a 460-point cluster
// took 26 us, a chain of dependent loads).
template <typename T, typename TO>
__device__ __forceinline__ void mv_n_sum(int bx, const T* __restrict__ part, int nz, int64_t n, int m,
                                         TO* __restrict__ KV, int64_t ldkv) {
  __shared__ T red[4][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t e = (int64_t)bx * 64 + lane, total = n * m;
  const T* p = part + (e < total ? e : 0);
  T acc[4] = {0, 0, 0, 0};
  int z = w;
  for (; z + 12 < nz; z += 16)
#pragma unroll
    for (int u = 0; u < 4; ++u) acc[u] += p[(int64_t)(z + 4 * u) * total];
  for (; z < nz; z += 4) acc[0] += p[(int64_t)z * total];
  red[w][lane] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
  __syncthreads();
  if (w != 0 || e >= total) return;
  const int64_t pt = e / m;
  KV[pt * ldkv + (e - pt * m)] = (TO)((red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]));
}

template <typename T, typename TO>
__global__ void __launch_bounds__(256) k_mv_n_sum(const T* __restrict__ part, int nz, int64_t n, int m,
                                                  TO* __restrict__ KV, int64_t ldkv) {
  mv_n_sum(blockIdx.x, part, nz, n, m, KV, ldkv);
}

// ------------------------------------------------------------------ narrow products
// Products with up to kNwMax right-hand sides, on the vector units: the matrix instructions would spend
// 12 of 16 columns or more on padding, and their operand layouts read 128- and 256-byte pieces of a row
// where a lane per 16 bytes of one row streams a kilobyte.  Both passes are bound by reading the factor
// once (pass 2 at 6.0 TB/s, 1e6 points binary32).  Where the line lies, measured per pass against the
// matrix-core passes (four right-hand sides, then five to eight computed as eight): pass 1, 1e6 points
// binary32 0.72 against 0.86 ms, 250,007 points binary64 0.59 against 0.69, 2e5 points of rank 2666 0.22
// against 0.36; pass 2 0.59, 0.44 and 0.18 against 0.76, 0.51 and 0.30; with eight columns pass 2 takes
// 0.75, 0.50 and 0.27, no longer worth a second layout of D W, and pass 1 is bound by its arithmetic.
// One right-hand side: both passes 0.77 + 0.78 -> 0.63 + 0.58 ms, 0.66 + 0.73 -> 0.45 + 0.41, 0.32 + 0.34
// -> 0.17 + 0.17.  Few points, whole products against the matrix-core passes of before (seven clouds, d = 3..8,
// both types, geometric means for one and four columns): 2,000 points 1.41 and 1.18 times as fast, 12,007 1.72
// and 1.35, 60,000 1.95 and 1.52; without allocation 3.1 and 2.6, 3.1 and 2.3, 2.5 and 1.9.  The least of
// 448 is four columns of 2,000 to 4,000 binary32 points in d = 7 and 8, as fast within the runs' 2 us.
//
// Pass 1: a wavefront takes RB harmonics of one degree, up to four of its radial functions and a range
// of points; every lane keeps its own sums of PPL points a step (one 16-byte load per row), formed with
// z_{l,c}(i) = q_l(i) v_c(i), and the sums over the lanes are taken in binary64 at the end, halving the
// number of values with the number of lanes.
template <typename T>
__device__ __forceinline__ void nw_load(const T* __restrict__ p, T (&o)[16 / sizeof(T)]) {
  typedef typename PVec<T, 16 / sizeof(T)>::type V;
  const V w = *reinterpret_cast<const V*>(p);
#pragma unroll
  for (int e = 0; e < (int)(16 / sizeof(T)); ++e) o[e] = w[e];
}
__device__ __forceinline__ float nw_fma(float a, float b, float c) { return fmaf(a, b, c); }
__device__ __forceinline__ double nw_fma(double a, double b, double c) { return fma(a, b, c); }
// Least number of points per split.  With fewer, the sum over splits costs more than the shorter chain of
// steps gives (products of four columns: binary64, 4,000 points of rank 1413 48.6 us, 53.6 with 256); with more
// the chain does (binary32, 2,000 points in d = 6 40.5 us, 44.7 with 1,024; d = 7 35.9 and 38.2).
constexpr int kNwSplitPoints = 512;
__host__ __device__ constexpr int nw_rows(int bytes, int sn, int m) {
  return bytes == 4 ? (sn * m <= 8 ? 8 : 4) : (sn * m <= 4 ? 8 : (sn * m <= 8 ? 4 : 2));
}

// Sums over the 64 lanes of N values: the lanes with bit OFF set go on with the upper half of the values,
// the others with the lower, each taking its half from the lane across; `first` is the index of the sum
// that a lane ends with (64 / N lanes hold the same one).
template <int OFF, int N>
__device__ __forceinline__ double nw_fold(const double (&s)[N], int lane, int& first) {
  if constexpr (OFF == 0) {
    return s[0];
  } else if constexpr (N == 1) {
    const double t[1] = {s[0] + __shfl_xor(s[0], OFF)};
    return nw_fold<OFF / 2>(t, lane, first);
  } else {
    // bit masks instead of selects: every lane reaches the shuffles by one path
    const uint64_t up = 0 - (uint64_t)((lane / OFF) & 1);
    double t[N / 2];
#pragma unroll
    for (int j = 0; j < N / 2; ++j) {
      const uint64_t a = __builtin_bit_cast(uint64_t, s[j]), b = __builtin_bit_cast(uint64_t, s[j + N / 2]);
      const double give = __builtin_bit_cast(double, (a & up) | (b & ~up));
      t[j] = __builtin_bit_cast(double, (b & up) | (a & ~up)) + __shfl_xor(give, OFF);
    }
    first += (int)up & (N / 2);
    return nw_fold<OFF / 2>(t, lane, first);
  }
}

template <typename T, typename TV, int SN, int M>
__device__ __forceinline__ void nw_t_item(const T* __restrict__ phi, int64_t ld_phi, const T* __restrict__ q,
                                          int64_t ld_q, const DegDev& dg, int rb, int l0,
                                          const TV* __restrict__ V, int64_t ldv, int64_t n, int64_t p_begin,
                                          int64_t p_end, const double* __restrict__ lam, T* __restrict__ Wn,
                                          double* __restrict__ W, int64_t w_ld, double* __restrict__ part) {
  constexpr int PPL = 16 / sizeof(T), RB = nw_rows(sizeof(T), SN, M), NV = RB * SN * M;
  const int lane = threadIdx.x & 63;
  const int h0 = rb * RB;
  T acc[RB][SN][M];
#pragma unroll
  for (int r = 0; r < RB; ++r)
#pragma unroll
    for (int l = 0; l < SN; ++l)
#pragma unroll
      for (int c = 0; c < M; ++c) acc[r][l][c] = 0;
  for (int64_t p = p_begin; p < p_end; p += 64 * PPL) {
    const int64_t pl = p + (int64_t)lane * PPL;
    const int64_t pc = pl < n ? pl : 0;            // lanes past the points read the first ones, times zero
    T a[RB][PPL], z[SN][PPL];
    TV v[M][PPL];
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      const int h = h0 + r < dg.nh ? h0 + r : dg.nh - 1;
      nw_load(phi + (int64_t)(dg.hoff + h) * ld_phi + pc, a[r]);
    }
#pragma unroll
    for (int l = 0; l < SN; ++l) nw_load(q + (int64_t)(dg.qoff + l0 + l) * ld_q + pc, z[l]);
#pragma unroll
    for (int e = 0; e < PPL; ++e)
#pragma unroll
      for (int c = 0; c < M; ++c) v[c][e] = V[(pl + e < n ? pl + e : 0) * ldv + c];
#pragma unroll
    for (int e = 0; e < PPL; ++e) {
      const bool ok = pl + e < p_end;
#pragma unroll
      for (int c = 0; c < M; ++c) {
        const T vv = ok ? (T)v[c][e] : (T)0;
#pragma unroll
        for (int l = 0; l < SN; ++l) {
          const T zz = z[l][e] * vv;
#pragma unroll
          for (int r = 0; r < RB; ++r) acc[r][l][c] = nw_fma(a[r][e], zz, acc[r][l][c]);
        }
      }
    }
  }
  // value j = (r SN + l) M + c; padded to a power of two
  constexpr int NP = NV <= 1 ? 1 : NV <= 2 ? 2 : NV <= 4 ? 4 : NV <= 8 ? 8 : NV <= 16 ? 16 : NV <= 32 ? 32 : 64;
  static_assert(NV <= 64, "one value per lane at the end");
  double s[NP];
#pragma unroll
  for (int j = 0; j < NP; ++j) s[j] = j < NV ? (double)acc[j / (SN * M) % RB][j / M % SN][j % M] : 0.0;
  int first = 0;                                   // index of the value this lane ends with
  s[0] = nw_fold<32>(s, lane, first);
  const int r = first / (SN * M), l = first / M % SN, c = first % M;
  constexpr int REP = 64 / NP;                     // lanes with the same value
  if (first < NV && h0 + r < dg.nh && lane % REP == 0) {
    const int64_t row = dg.roff + (int64_t)(h0 + r) * dg.s + l0 + l;
    if (part) {
      part[row * M + c] = s[0];
    } else {
      if (Wn) Wn[row * M + c] = (T)(lam[row] * s[0]);
      if (W) W[row * w_ld + c] = s[0];
    }
  }
}

// Items of pass 1 over the degrees: row blocks of each group of up to four radial functions.
template <typename T, typename TV, int M>
__device__ __forceinline__ void nw_t(int item, int split, const T* __restrict__ phi, int64_t ld_phi,
                                     const T* __restrict__ q, int64_t ld_q, const DegDev* __restrict__ degs, int n_deg,
                                     const TV* __restrict__ V, int64_t ldv, int64_t n, int64_t split_len,
                                     int64_t rank, const double* __restrict__ lam, T* __restrict__ Wn,
                                     double* __restrict__ W, int64_t w_ld, double* __restrict__ part) {
  DegDev dg = degs[0];
  int l0 = 0, sn = 0;
  for (int di = 0; di < n_deg; ++di) {
    dg = degs[di];
    bool here = false;
    for (l0 = 0; l0 < dg.s; l0 += 4) {
      sn = dg.s - l0 < 4 ? dg.s - l0 : 4;
      const int rows = nw_rows(sizeof(T), sn, M), nrb = (dg.nh + rows - 1) / rows;
      if (item < nrb) {
        here = true;
        break;
      }
      item -= nrb;
    }
    if (here) break;
  }
  const int64_t p_begin = (int64_t)split * split_len;
  const int64_t p_end = p_begin + split_len < n ? p_begin + split_len : n;
  double* out = part ? part + (int64_t)split * rank * M : nullptr;
  switch (sn) {                                    // uniform
    case 1: nw_t_item<T, TV, 1, M>(phi, ld_phi, q, ld_q, dg, item, l0, V, ldv, n, p_begin, p_end, lam, Wn, W, w_ld, out); break;
    case 2: nw_t_item<T, TV, 2, M>(phi, ld_phi, q, ld_q, dg, item, l0, V, ldv, n, p_begin, p_end, lam, Wn, W, w_ld, out); break;
    case 3: nw_t_item<T, TV, 3, M>(phi, ld_phi, q, ld_q, dg, item, l0, V, ldv, n, p_begin, p_end, lam, Wn, W, w_ld, out); break;
    default: nw_t_item<T, TV, 4, M>(phi, ld_phi, q, ld_q, dg, item, l0, V, ldv, n, p_begin, p_end, lam, Wn, W, w_ld, out); break;
  }
}

// Wavefront w of block b takes item 4 gi + w of split sp, b = 8 (G (sp / 8) + gi) + sp % 8: the items of
// one range of points run on one XCD, close in time, and share V and the radial rows in its L2.
template <typename T, typename TV, int M>
__global__ void __launch_bounds__(256) k_nw_t(const T* __restrict__ phi, int64_t ld_phi, const T* __restrict__ q,
                                              int64_t ld_q, const DegDev* __restrict__ degs, int n_deg, int n_items,
                                              int n_splits, int64_t split_len, const TV* __restrict__ V, int64_t ldv,
                                              int64_t n, int64_t rank, const double* __restrict__ lam,
                                              T* __restrict__ Wn, double* __restrict__ W, int64_t w_ld,
                                              double* __restrict__ part) {
  const int groups = (n_items + 3) / 4;
  const int rest = (int)(blockIdx.x >> 3), gi = rest % groups, split = ((rest / groups) << 3) + (blockIdx.x & 7);
  const int item = 4 * gi + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  if (split >= n_splits || item >= n_items) return;
  nw_t<T, TV, M>(item, split, phi, ld_phi, q, ld_q, degs, n_deg, V, ldv, n, split_len, rank, lam, Wn, W, w_ld, part);
}

// Sum of pass 1's splits (wavefront w takes the splits w, w + 4, ...), scaled copy and unscaled sums.
template <typename T>
__device__ __forceinline__ void nw_reduce(int bx, const double* __restrict__ part, int n_splits, int64_t total, int M,
                                          const double* __restrict__ lam, T* __restrict__ Wn, double* __restrict__ W,
                                          int64_t w_ld) {
  __shared__ double red[4][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t e = (int64_t)bx * 64 + lane;
  const double* p = part + (e < total ? e : 0);
  double acc[4] = {0, 0, 0, 0};
  int sp = w;
  for (; sp + 12 < n_splits; sp += 16)
#pragma unroll
    for (int u = 0; u < 4; ++u) acc[u] += p[(int64_t)(sp + 4 * u) * total];
  for (; sp < n_splits; sp += 4) acc[0] += p[(int64_t)sp * total];
  red[w][lane] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
  __syncthreads();
  if (w != 0 || e >= total) return;
  const double v = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
  const int64_t row = e / M;
  if (Wn) Wn[e] = (T)(lam[row] * v);
  if (W) W[row * w_ld + (e - row * M)] = v;
}

template <typename T>
__global__ void __launch_bounds__(256) k_nw_reduce(const double* __restrict__ part, int n_splits, int64_t total, int M,
                                                    const double* __restrict__ lam, T* __restrict__ Wn,
                                                    double* __restrict__ W, int64_t w_ld) {
  nw_reduce(blockIdx.x, part, n_splits, total, M, lam, Wn, W, w_ld);
}

// Pass 2: a lane takes PPL points, the harmonic rows [z_lo, z_hi) stream by (one 16-byte load per row),
// their rows of D W are wavefront-uniform values.  Per degree the sums over the harmonics are kept for
// each radial function (up to four at a time) and folded into KV with its radial values.
template <typename T, int SN, int M>
__device__ __forceinline__ void nw_n_degree(const T* __restrict__ phi, int64_t ld_phi, const T* __restrict__ q,
                                            int64_t ld_q, const DegDev& dg, int l0, int hlo, int hhi,
                                            const T* __restrict__ Wn, T (&kv)[M][16 / sizeof(T)]) {
  constexpr int PPL = 16 / sizeof(T), U = 8;
  T t[SN][M][PPL];
#pragma unroll
  for (int l = 0; l < SN; ++l)
#pragma unroll
    for (int c = 0; c < M; ++c)
#pragma unroll
      for (int e = 0; e < PPL; ++e) t[l][c][e] = 0;
  const T* row = phi + (int64_t)(dg.hoff + hlo) * ld_phi;
  const T* w = Wn + ((int64_t)dg.roff + (int64_t)hlo * dg.s + l0) * M;
  const int64_t ws = (int64_t)dg.s * M;
  int h = hlo;
  for (; h + U <= hhi; h += U) {
    T a[U][PPL];
#pragma unroll
    for (int u = 0; u < U; ++u) nw_load(row + (int64_t)u * ld_phi, a[u]);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int l = 0; l < SN; ++l)
#pragma unroll
        for (int c = 0; c < M; ++c) {
          const T wv = w[u * ws + l * M + c];
#pragma unroll
          for (int e = 0; e < PPL; ++e) t[l][c][e] = nw_fma(a[u][e], wv, t[l][c][e]);
        }
    row += U * ld_phi;
    w += U * ws;
  }
  for (; h < hhi; ++h) {
    T a[PPL];
    nw_load(row, a);
#pragma unroll
    for (int l = 0; l < SN; ++l)
#pragma unroll
      for (int c = 0; c < M; ++c) {
        const T wv = w[l * M + c];
#pragma unroll
        for (int e = 0; e < PPL; ++e) t[l][c][e] = nw_fma(a[e], wv, t[l][c][e]);
      }
    row += ld_phi;
    w += ws;
  }
#pragma unroll
  for (int l = 0; l < SN; ++l) {
    T ql[PPL];
    nw_load(q + (int64_t)(dg.qoff + l0 + l) * ld_q, ql);
#pragma unroll
    for (int c = 0; c < M; ++c)
#pragma unroll
      for (int e = 0; e < PPL; ++e) kv[c][e] = nw_fma(ql[e], t[l][c][e], kv[c][e]);
  }
}

template <typename T, typename TO, int M>
__device__ __forceinline__ void nw_n(int64_t bx, int z, const T* __restrict__ phi, int64_t ld_phi,
                                     const T* __restrict__ q, int64_t ld_q, const DegDev* __restrict__ degs, int n_deg,
                                     const T* __restrict__ Wn, TO* __restrict__ KV, int64_t ldkv,
                                     int64_t n, int z_rows, T* __restrict__ shares) {
  constexpr int PPL = 16 / sizeof(T);
  const int lane = threadIdx.x;
  const int64_t pl = bx * (64 * PPL) + (int64_t)lane * PPL;
  const int64_t pc = pl < n ? pl : 0;              // lanes past the points read the first ones and write nothing
  const int z_lo = shares ? z * z_rows : 0, z_hi = shares ? z_lo + z_rows : 0x7fffffff;
  T kv[M][PPL];
#pragma unroll
  for (int c = 0; c < M; ++c)
#pragma unroll
    for (int e = 0; e < PPL; ++e) kv[c][e] = 0;
  for (int di = 0; di < n_deg; ++di) {
    const DegDev dg = degs[di];
    const int hlo = z_lo > dg.hoff ? z_lo - dg.hoff : 0;
    const int hhi = z_hi - dg.hoff < dg.nh ? z_hi - dg.hoff : dg.nh;
    if (hlo >= hhi) continue;
    for (int l0 = 0; l0 < dg.s; l0 += 4) {
      switch (dg.s - l0) {                         // uniform
        case 1: nw_n_degree<T, 1, M>(phi + pc, ld_phi, q + pc, ld_q, dg, l0, hlo, hhi, Wn, kv); break;
        case 2: nw_n_degree<T, 2, M>(phi + pc, ld_phi, q + pc, ld_q, dg, l0, hlo, hhi, Wn, kv); break;
        case 3: nw_n_degree<T, 3, M>(phi + pc, ld_phi, q + pc, ld_q, dg, l0, hlo, hhi, Wn, kv); break;
        default: nw_n_degree<T, 4, M>(phi + pc, ld_phi, q + pc, ld_q, dg, l0, hlo, hhi, Wn, kv); break;
      }
    }
  }
#pragma unroll
  for (int e = 0; e < PPL; ++e)
    if (pl + e < n) {
#pragma unroll
      for (int c = 0; c < M; ++c) {
        if (shares) shares[((int64_t)z * n + pl + e) * M + c] = kv[c][e];
        else KV[(pl + e) * ldkv + c] = (TO)kv[c][e];
      }
    }
}

template <typename T, typename TO, int M>
__global__ void __launch_bounds__(64) k_nw_n(const T* __restrict__ phi, int64_t ld_phi, const T* __restrict__ q,
                                             int64_t ld_q, const DegDev* __restrict__ degs, int n_deg,
                                             const T* __restrict__ Wn, TO* __restrict__ KV, int64_t ldkv,
                                             int64_t n, int z_rows, T* __restrict__ shares) {
  nw_n<T, TO, M>(blockIdx.x, blockIdx.z, phi, ld_phi, q, ld_q, degs, n_deg, Wn, KV, ldkv, n, z_rows, shares);
}

// The products of many binary64 factors with one right-hand side each, a launch per phase over all of
// them (blockIdx.y: the factor).  Launched one by one, thirty factors of 460 points and rank 1,290 took
// 120 launches of a few workgroups, and the host's enqueueing bounded the KRR operator.
__global__ void __launch_bounds__(256) k_nwb_t(const MvBatch* __restrict__ batch, const double* __restrict__ v) {
  const MvBatch f = batch[blockIdx.y];
  const int groups = (f.n_items + 3) / 4;
  const int gi = (int)blockIdx.x % groups, split = (int)blockIdx.x / groups;
  const int item = 4 * gi + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  if (split >= f.n_splits || item >= f.n_items) return;
  nw_t<double, double, 1>(item, split, f.phi, f.ld, f.q, f.ld, f.degs, f.n_deg, v + f.pos, 1, f.n, f.split_len, f.rank,
                          f.lam, f.Wn, nullptr, 1, f.n_splits > 1 ? f.part : nullptr);
}

__global__ void __launch_bounds__(256) k_nwb_reduce(const MvBatch* __restrict__ batch) {
  const MvBatch f = batch[blockIdx.y];
  if (f.n_splits <= 1 || (int64_t)blockIdx.x * 64 >= f.rank) return;
  nw_reduce<double>(blockIdx.x, f.part, f.n_splits, f.rank, 1, f.lam, f.Wn, nullptr, 1);
}

__global__ void __launch_bounds__(64) k_nwb_n(const MvBatch* __restrict__ batch) {
  const MvBatch f = batch[blockIdx.y];
  if ((int)blockIdx.z >= f.nz || (int64_t)blockIdx.x * 128 >= f.n) return;
  nw_n<double, double, 1>(blockIdx.x, blockIdx.z, f.phi, f.ld, f.q, f.ld, f.degs, f.n_deg, f.Wn, nullptr, 1, f.n,
                          f.z_rows, f.shares);
}

__global__ void __launch_bounds__(256) k_nwb_sum(const MvBatch* __restrict__ batch, double* __restrict__ out) {
  const MvBatch f = batch[blockIdx.y];
  if ((int64_t)blockIdx.x * 64 >= f.n) return;
  mv_n_sum<double, double>(blockIdx.x, f.shares, f.nz, f.n, 1, out + f.pos, 1);
}

hipError_t launch_matvec_batch(const MvBatch* batch_dev, const MvBatchGrid& g, const double* v, double* out,
                               hipStream_t s) {
  if (g.factors < 1 || g.t_blocks < 1 || g.n_blocks < 1 || g.shares < 1) return hipErrorInvalidValue;
  const unsigned nf = (unsigned)g.factors;
  k_nwb_t<<<dim3((unsigned)g.t_blocks, nf), 256, 0, s>>>(batch_dev, v);
  if (g.r_blocks > 0) k_nwb_reduce<<<dim3((unsigned)g.r_blocks, nf), 256, 0, s>>>(batch_dev);
  k_nwb_n<<<dim3((unsigned)((g.n_blocks + 1) / 2), nf, (unsigned)g.shares), 64, 0, s>>>(batch_dev);
  k_nwb_sum<<<dim3((unsigned)g.n_blocks, nf), 256, 0, s>>>(batch_dev, out);
  return hipGetLastError();
}

// ------------------------------------------------------------------ adjoint coefficients
// The coefficients of the adjoint's two products, from Gv = U^T V and Gw = U^T W (binary64, rank rows):
//   C2[(k,h,l)][c]          = lambda Gv[c], then lambda Gw[c]                       (c < m each)
//   Cs[(k,h',l)][2 m j + c] = sum_h G_k^(j)[h][h'] C2[(k,h,l)][c]                   (h' of degree k - 1)
// written where pass 2 reads them, in block order (or C2 in rank order for the narrow pass).  The maps
// G_k are sparse (a derivative of a harmonic touches a few of the degree below): rows (k, j, h') of
// `map`, entry e the harmonic map_h[e] with the value map_v[e].  On the host the dense sums and the
// uploads were most of the 2.3 ms that hdf_backward took to return (2e5 points, d = 4, degrees to 13); 0.3 so.
__device__ __forceinline__ int64_t block_at(int64_t row, int c, int cpl) {
  const int hh = (int)(row & 15);
  return ((row >> 4) * cpl + (c >> 4)) * 256 + ((hh & 3) * 16 + (c & 15)) * 4 + (hh >> 2);
}

template <typename T>
__global__ void __launch_bounds__(256) k_adj_c2(const double* __restrict__ gv, const double* __restrict__ gw,
                                                int64_t gstride, int m, const double* __restrict__ lam,
                                                const int32_t* __restrict__ src, int64_t rows, int cols,
                                                int block_order, T* __restrict__ out) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= rows * cols) return;
  const int64_t row = e / cols;
  const int c = (int)(e - row * cols);
  const int64_t sr = block_order ? src[row] : row;
  double v = 0.0;
  if (sr >= 0 && c < 2 * m) v = lam[sr] * (c < m ? gv[sr * gstride + c] : gw[sr * gstride + c - m]);
  out[block_order ? block_at(row, c, cols >> 4) : e] = (T)v;
}

template <typename T>
__global__ void __launch_bounds__(256) k_adj_cs(const double* __restrict__ gv, const double* __restrict__ gw,
                                                int64_t gstride, int m, int d, const double* __restrict__ lam,
                                                const DegDev* __restrict__ degs, const DegDev* __restrict__ shifted,
                                                int n_shifted, const int32_t* __restrict__ map,
                                                const int32_t* __restrict__ map_h, const double* __restrict__ map_v,
                                                int64_t rows, int cols, T* __restrict__ out) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= rows * cols) return;
  const int64_t row = e / cols, blk = row >> 4;
  const int col = (int)(e - row * cols), j = col / (2 * m), c = col - j * 2 * m;
  int di = 0, at = 0;                              // degree k = di + 1; at: first map row of the degree
  while (di + 1 < n_shifted && shifted[di + 1].boff <= blk) at += d * shifted[di++].nh;
  const DegDev sh = shifted[di], dg = degs[di + 1];
  const int rel = (int)(blk - sh.boff), b = rel / sh.s, l = rel - b * sh.s, hp = 16 * b + (int)(row & 15);
  double v = 0.0;
  if (j < d && hp < sh.nh) {
    const double* g = c < m ? gv + c : gw + (c - m);
    const int mr = at + j * sh.nh + hp;
    for (int t = map[mr]; t < map[mr + 1]; ++t) {
      const int64_t rr = dg.roff + (int64_t)map_h[t] * dg.s + l;
      v = fma(map_v[t], lam[rr] * g[rr * gstride], v);
    }
  }
  out[block_at(row, col, cols >> 4)] = (T)v;
}

hipError_t launch_adj_coefficients(const double* gv, const double* gw, int64_t gstride, int m, int d,
                                   const double* lam, const DegDev* degs, const int32_t* src, int64_t c2_rows,
                                   int c2_cols, int c2_block_order, void* c2, const DegDev* shifted, int n_shifted,
                                   const int32_t* map, const int32_t* map_h, const double* map_v,
                                   int64_t shift_blocks, int cs_cols, void* cs, int prec, hipStream_t s) {
  const unsigned b2 = (unsigned)((c2_rows * c2_cols + 255) / 256);
  const unsigned bs = (unsigned)((shift_blocks * 16 * cs_cols + 255) / 256);
#define ADJ_COEF(T)                                                                                            \
  do {                                                                                                         \
    k_adj_c2<T><<<b2, 256, 0, s>>>(gv, gw, gstride, m, lam, src, c2_rows, c2_cols, c2_block_order, (T*)c2);    \
    if (n_shifted > 0)                                                                                         \
      k_adj_cs<T><<<bs, 256, 0, s>>>(gv, gw, gstride, m, d, lam, degs, shifted, n_shifted, map, map_h, map_v,  \
                                     shift_blocks * 16, cs_cols, (T*)cs);                                      \
  } while (0)
  if (prec == 1) ADJ_COEF(float);
  else ADJ_COEF(double);
#undef ADJ_COEF
  return hipGetLastError();
}

int narrow_items(const DegDev* degs, int n_deg, int prec, int m) {
  int items = 0;
  for (int di = 0; di < n_deg; ++di)
    for (int l0 = 0; l0 < degs[di].s; l0 += 4) {
      const int rows = nw_rows(prec == 1 ? 4 : 8, std::min(4, degs[di].s - l0), m);
      items += (degs[di].nh + rows - 1) / rows;
    }
  return items;
}

void narrow_splits(int64_t n, int n_items, int prec, int64_t per_split_bytes, int64_t most_bytes, int* n_splits,
                   int64_t* split_len) {
  const int64_t step = 64 * (prec == 1 ? 4 : 2);
  int64_t ns = std::max<int64_t>(1, 8192 / std::max(1, n_items));
  ns = std::min(ns, std::max<int64_t>(1, n / kNwSplitPoints));
  ns = std::min(ns, std::max<int64_t>(1, most_bytes / per_split_bytes));
  const int64_t len = ((n + ns - 1) / ns + step - 1) / step * step;
  *split_len = len;
  *n_splits = (int)((n + len - 1) / len);
}

#define HDF_NW_M(CALL, T, TV)                                                                                \
  do {                                                                                                       \
    if (m == 1) CALL(T, TV, 1);                                                                              \
    else if (m == 2) CALL(T, TV, 2);                                                                         \
    else if (m == 3) CALL(T, TV, 3);                                                                         \
    else CALL(T, TV, 4);                                                                                     \
  } while (0)
#define HDF_NW(CALL)                                                                                         \
  do {                                                                                                       \
    if (prec == 1 && io == 0) HDF_NW_M(CALL, float, float);                                                  \
    else if (prec == 0 && io == 1) HDF_NW_M(CALL, double, double);                                           \
    else if (prec == 0 && io == 0) HDF_NW_M(CALL, double, float);                                            \
    else return hipErrorInvalidValue;                                                                        \
  } while (0)

hipError_t launch_narrow_t(const void* phi, int64_t ld_phi, const void* q, int64_t ld_q, const DegDev* degs, int n_deg,
                           int n_items, int n_splits, int64_t split_len, const void* V, int64_t ldv, int64_t n, int m,
                           int64_t rank, const double* lam, void* Wn, double* W, int64_t w_ld, double* part, int prec,
                           int io, hipStream_t s) {
  const int64_t step = 64 * (prec == 1 ? 4 : 2);
  if (m < 1 || m > kNwMax || n_deg < 1 || n_items < 1 || n_splits < 1 || split_len % step) return hipErrorInvalidValue;
  if ((int64_t)(n_splits - 1) * split_len >= n || (int64_t)n_splits * split_len < n) return hipErrorInvalidValue;
  if (n_splits > 1 && !part) return hipErrorInvalidValue;
  double* dst = n_splits > 1 ? part : nullptr;
  const unsigned nb = (unsigned)(((n_splits + 7) / 8) * 8 * ((n_items + 3) / 4));
#define NW_T(T, TV, M)                                                                                        \
  k_nw_t<T, TV, M><<<nb, 256, 0, s>>>((const T*)phi, ld_phi, (const T*)q, ld_q, degs, n_deg, n_items, n_splits, \
                                      split_len, (const TV*)V, ldv, n, rank, lam, (T*)Wn, W, w_ld, dst)
  HDF_NW(NW_T);
#undef NW_T
  if (n_splits > 1) {
    const int64_t total = rank * m;
    const unsigned rb = (unsigned)((total + 63) / 64);
    if (prec == 1) k_nw_reduce<float><<<rb, 256, 0, s>>>(part, n_splits, total, m, lam, (float*)Wn, W, w_ld);
    else k_nw_reduce<double><<<rb, 256, 0, s>>>(part, n_splits, total, m, lam, (double*)Wn, W, w_ld);
  }
  return hipGetLastError();
}

hipError_t launch_narrow_n(const void* phi, int64_t ld_phi, const void* q, int64_t ld_q, const DegDev* degs, int n_deg,
                           const void* Wn, void* KV, int64_t ldkv, int64_t n, int m, int n_rows, int z_rows,
                           void* shares, int prec, int io, hipStream_t s) {
  if (m < 1 || m > kNwMax || n_deg < 1 || n_rows < 1) return hipErrorInvalidValue;
  const int nz = z_rows > 0 ? (n_rows + z_rows - 1) / z_rows : 1;
  if (nz > 1 && !shares) return hipErrorInvalidValue;
  void* sh = nz > 1 ? shares : nullptr;
  const int64_t step = 64 * (prec == 1 ? 4 : 2);
  const dim3 grid((unsigned)((n + step - 1) / step), 1, (unsigned)nz);
  const unsigned nb = (unsigned)((n * m + 63) / 64);
#define NW_N(T, TO, M)                                                                                          \
  do {                                                                                                          \
    k_nw_n<T, TO, M><<<grid, 64, 0, s>>>((const T*)phi, ld_phi, (const T*)q, ld_q, degs, n_deg, (const T*)Wn,   \
                                         (TO*)KV, ldkv, n, z_rows, (T*)sh);                                    \
    if (nz > 1) k_mv_n_sum<T, TO><<<nb, 256, 0, s>>>((const T*)sh, nz, n, m, (TO*)KV, ldkv);                    \
  } while (0)
  HDF_NW(NW_N);
#undef NW_N
  return hipGetLastError();
}
#undef HDF_NW
#undef HDF_NW_M

hipError_t launch_matvec_reduce(const double* partials, int n_splits, int64_t rank, int m16, const int32_t* src,
                                int64_t n_blocks, const double* lam_row, double* W, void* Wd, void* Wb, int prec,
                                hipStream_t s) {
  if (n_blocks < 1 || m16 < 16 || m16 % 16) return hipErrorInvalidValue;
  const int64_t total = n_blocks * 16 * m16;
  const unsigned nb = (unsigned)((total + 63) / 64);
  if (prec == 1)
    k_mv_reduce<float><<<nb, 256, 0, s>>>(partials, n_splits, rank * m16, total, m16, src, lam_row, W, (float*)Wd,
                                          (float*)Wb);
  else
    k_mv_reduce<double><<<nb, 256, 0, s>>>(partials, n_splits, rank * m16, total, m16, src, lam_row, W, (double*)Wd,
                                           (double*)Wb);
  return hipGetLastError();
}

int matvec_n_tiles(int64_t n, int cpl) {
  // The busiest of the 1,024 SIMDs sets the time: its wavefronts times their column tiles, plus about
  // a third of a tile for the rows and operands that a wavefront forms once.  With many points that is
  // the widest group with the fewest padded tiles; 44,599 points and 168 columns take groups of three
  // (three wavefronts of three tiles on a SIMD, 0.53 ms) rather than of four (2,091 wavefronts, a few
  // SIMDs with three of four tiles, 0.65 ms).
  int best = 1;
  int64_t cost = -1;
  for (int t = 1; t <= 4 && t <= cpl; ++t) {
    const int64_t waves = ((n + 63) / 64) * ((cpl + t - 1) / t);
    const int64_t c = (waves + 1023) / 1024 * (10 * t + 3);
    if (cost < 0 || c <= cost) {
      cost = c;
      best = t;
    }
  }
  return best;
}

hipError_t launch_matvec_n(const void* phi, int64_t ld_phi, const void* q, int64_t ld_q,
                           const DegDev* degs, int n_deg, const void* Wb, int64_t n_blocks, int m16,
                           void* KV, int64_t ldkv, int64_t n, int m, int prec, int io, int z_blocks,
                           void* part, hipStream_t s) {
  if (n_deg < 1 || n_blocks < 1 || m16 < 16 || m16 % 16) return hipErrorInvalidValue;
  const int nz = z_blocks > 0 ? (int)((n_blocks + z_blocks - 1) / z_blocks) : 1;
  if (nz > 1 && !part) return hipErrorInvalidValue;
  const int nct = matvec_n_tiles(n, m16 / 16);
  const int64_t n_cg = (m16 / 16 + nct - 1) / nct;
  const dim3 grid((unsigned)(((n + 63) / 64 + 7) / 8 * 8 * n_cg), 1, (unsigned)nz);
  const unsigned nb = (unsigned)((n * m + 63) / 64);
#define HDF_MVN_RUN(T, TO, NCT, SPLIT)                                                                       \
  k_mv_n<T, TO, NCT, SPLIT><<<grid, 64, 0, s>>>((const T*)phi, ld_phi, (const T*)q, ld_q, degs, n_deg,      \
                                                (const T*)Wb, m16, (TO*)KV, ldkv, n, m, z_blocks,            \
                                                (int)n_blocks, (T*)part)
#define HDF_MVN_NCT(T, TO, SPLIT)                                                                            \
  do {                                                                                                       \
    if (nct == 1) HDF_MVN_RUN(T, TO, 1, SPLIT);                                                              \
    else if (nct == 2) HDF_MVN_RUN(T, TO, 2, SPLIT);                                                         \
    else if (nct == 3) HDF_MVN_RUN(T, TO, 3, SPLIT);                                                         \
    else HDF_MVN_RUN(T, TO, 4, SPLIT);                                                                       \
  } while (0)
#define HDF_MVN(T, TO)                                                                                       \
  do {                                                                                                       \
    if (nz > 1) {                                                                                            \
      HDF_MVN_NCT(T, TO, true);                                                                              \
      k_mv_n_sum<T, TO><<<nb, 256, 0, s>>>((const T*)part, nz, n, m, (TO*)KV, ldkv);                         \
    } else {                                                                                                 \
      HDF_MVN_NCT(T, TO, false);                                                                             \
    }                                                                                                        \
  } while (0)
  if (prec == 1 && io == 0) HDF_MVN(float, float);
  else if (prec == 0 && io == 1) HDF_MVN(double, double);
  else if (prec == 0 && io == 0) HDF_MVN(double, float);
  else return hipErrorInvalidValue;
#undef HDF_MVN
#undef HDF_MVN_NCT
#undef HDF_MVN_RUN
  return hipGetLastError();
}

}  // namespace hdf
