// Cross tests: cross-MMD (Alg. 6) and cross-ED (Alg. 7) of the paper's appendix.
//
// x is cut into x1 (its first floor(nx/2) rows) and x2, y into y1 and y2.  The block stage
// runs on the "x side" [x1; y1] against the "y side" [x2; y2] (the four cross blocks form
// that rectangle) and leaves, per tile and x-side row, the row's sums over the x2 columns
// and over the y2 columns.  Here, per x-side row a, with row means m2(a) over x2 and
// m3(a) over y2:
//   v(a) = m3(a) - m2(a) (ED)  or  m2(a) - m3(a) (MMD),
// so that U_x = mean of v over the x1 rows and U_y = mean of v over the y1 rows are the
// algorithms' differences of block means (a block mean is the mean of its row means);
//   U = U_x - U_y,  s_x = mean over x1 rows of (v - U_x)^2,  s_y likewise over y1 rows,
//   sigma = sqrt(s_x / |x1| + s_y / |y1|),  p = 1 - Phi(U / sigma) = erfc(z / sqrt 2) / 2.
// sigma = 0 gives z = +inf, -inf or 0 by the sign of U.  All sums are FP64 with
// compensation.
#include "common.h"

namespace et {

namespace {
struct Csum {  // compensated FP64 sum (Neumaier)
  double s = 0.0, c = 0.0;
  __device__ void add(double x) {
    const double t = s + x;
    c += fabs(s) >= fabs(x) ? (s - t) + x : (x - t) + s;
    s = t;
  }
  __device__ double value() const { return s + c; }
};
}  // namespace

// CF_WGS: one workgroup per x-side tile up to 16, then several tiles each.  Whole cross tests with
// 1 / 16 / 32 workgroups, FP32 form, p = 50: 100 + 100 rows (one tile) 52 / 52 / 53 us, 2000 +
// 2000 96 / 58 / 58, 4000 + 4000 162 / 81 / 78, 6000 + 6000 304 / 122 / 118; FP64 44 / 44 / 44,
// 116 / 77 / 77, 328 / 190 / 185, 645 / 362 / 356.
constexpr int CF_THREADS = 1024, CF_WGS = 16, CF_BATCH = 4;

// Workgroup-wide sums of two values (every thread returns them).
__device__ inline void block_sum2(double& a, double& b, double (*red)[CF_THREADS / 64]) {
  for (int m = 32; m > 0; m >>= 1) {
    a += __shfl_xor(a, m, 64);
    b += __shfl_xor(b, m, 64);
  }
  const int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) {
    red[0][w] = a;
    red[1][w] = b;
  }
  __syncthreads();
  a = 0.0;
  b = 0.0;
  for (int k = 0; k < CF_THREADS / 64; ++k) {
    a += red[0][k];
    b += red[1][k];
  }
}

// The x-side tiles are spread over CF_WGS workgroups: eight threads per row, thread q adding the
// sums of the column tiles q, q + 8, ... (FP64: two column halves each), CF_BATCH loaded at a
// time; the eight are then added in order.  The last workgroup to finish forms the statistic.
// One workgroup alone read the 512 KB of sums of a 2000 + 2000 test at 30 GB/s: 19 us, now 10.
__global__ void __launch_bounds__(CF_THREADS) k_cross_final(const TestDesc* __restrict__ descs) {
  __shared__ double red[2][CF_THREADS / 64];
  __shared__ double part[4][CF_THREADS];
  __shared__ int last;
  const TestDesc d = descs[0];
  const int64_t n_side = d.nx;  // x-side rows: x1 then y1
  const int64_t nx1 = d.cnx1, ny1 = d.cny1, nx2 = d.cnx2, ny2 = (int64_t)d.ny - d.cnx2;
  const bool ed = d.kind == KIND_ED, f64 = d.prec == PREC_F64;
  double* v = d.rsum;  // v(a) of every x-side row
  for (int64_t i = blockIdx.x; i < d.tx; i += CF_WGS) {
    const int r = threadIdx.x & (TILE - 1), q = threadIdx.x >> 7;
    Csum s2, s3;
    const int per = f64 ? 2 : 1, n = per * d.ty;
    const double* ts = d.tsum + i * d.ty * d.tsum_stride + r;
    for (int k0 = q; k0 < n; k0 += 8 * CF_BATCH) {
      double x[CF_BATCH], y[CF_BATCH];
#pragma unroll
      for (int u = 0; u < CF_BATCH; ++u) {
        const int k = min(k0 + 8 * u, n - 1);
        const double* t = ts + (int64_t)(k / per) * d.tsum_stride + (k % per) * TILE;
        x[u] = t[0];
        y[u] = t[per * TILE];
      }
#pragma unroll
      for (int u = 0; u < CF_BATCH; ++u)
        if (k0 + 8 * u < n) {
          s2.add(x[u]);
          s3.add(y[u]);
        }
    }
    part[0][threadIdx.x] = s2.s;
    part[1][threadIdx.x] = s2.c;
    part[2][threadIdx.x] = s3.s;
    part[3][threadIdx.x] = s3.c;
    __syncthreads();
    const int64_t a = i * TILE + r;
    if (q == 0 && a < n_side) {
#pragma unroll
      for (int k = 1; k < 8; ++k) {
        s2.add(part[0][k * TILE + r]);
        s2.c += part[1][k * TILE + r];
        s3.add(part[2][k * TILE + r]);
        s3.c += part[3][k * TILE + r];
      }
      const double m2 = s2.value() / (double)nx2, m3 = s3.value() / (double)ny2;
      __hip_atomic_store(v + a, ed ? m3 - m2 : m2 - m3, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
  }
  // v is stored and loaded past the XCDs' caches (agent scope): every wave waits for its own
  // stores, and no wave but the first has to write back or drop its cache (a fence in all 16
  // waves of 32 workgroups took 10 us)
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (threadIdx.x == 0)
    last = __hip_atomic_fetch_add(d.flags + FLAG_COUNT, 1, __ATOMIC_ACQ_REL,
                                  __HIP_MEMORY_SCOPE_AGENT) == CF_WGS - 1;
  __syncthreads();
  if (!last) return;
  auto at = [&](int64_t a) {
    return __hip_atomic_load(v + a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  Csum sx, sy;
  for (int64_t a = threadIdx.x; a < n_side; a += CF_THREADS) {
    const double x = at(a);
    if (a < 4 * CF_THREADS) (&part[0][0])[a] = x;  // for its own thread, below
    if (a < nx1) sx.add(x);
    else sy.add(x);
  }
  double tx = sx.value(), ty = sy.value();
  block_sum2(tx, ty, red);
  const double ux = tx / (double)nx1, uy = ty / (double)ny1;
  Csum qx, qy;
  for (int64_t a = threadIdx.x; a < n_side; a += CF_THREADS) {
    const double dev = (a < 4 * CF_THREADS ? (&part[0][0])[a] : at(a)) - (a < nx1 ? ux : uy);
    if (a < nx1) qx.add(dev * dev);
    else qy.add(dev * dev);
  }
  double vx = qx.value(), vy = qy.value();
  block_sum2(vx, vy, red);
  if (threadIdx.x == 0) {
    const double u = ux - uy;
    const double sigma = sqrt((vx / (double)nx1) / (double)nx1 + (vy / (double)ny1) / (double)ny1);
    double z;
    if (sigma > 0.0) z = u / sigma;
    else z = u > 0.0 ? INFINITY : (u < 0.0 ? -INFINITY : 0.0);
    d.out6[0] = u;
    d.out6[1] = sigma;
    d.out6[2] = z;
    d.out6[3] = 0.5 * erfc(z * 0.70710678118654752440);
    ((int2*)d.out6)[4] = make_int2(d.flags[0], d.flags[1]);
  }
}

void launch_cross_final(hipStream_t st, const TestDesc* d) {
  hipLaunchKernelGGL(k_cross_final, dim3(CF_WGS), dim3(CF_THREADS), 0, st, d);
}

}  // namespace et
