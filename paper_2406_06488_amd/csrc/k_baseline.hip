// The two baselines the efficient test is measured against, on the same chip:
//  - the standard permutation test (Alg. 4): every split's statistic recomputed from
//    distance (or kernel) blocks of its own X*, Y*;
//  - the pre-computation test (Alg. 5): the distance (kernel) matrix of the pooled sample
//    once, then per split the sums of the entries its index sets select.
// Both count exceedances against the identity split evaluated by their own code, as the
// efficient test does: p = (1 + #{b < B : stat*_b >= stat_B}) / (1 + B).
#include "common.h"

#include <algorithm>

namespace et {

// ------------------------------------------------------------------ standard test
// Row map of split b: pooled items of x* in increasing order, then those of y* -- the
// index sets i*_x, i*_y of Alg. 4 -- so that the Gram reads X* and Y* through the map from rows
// that were staged once.
// One workgroup per split; maps k >= count are the identity (the observed split).
// Every member word holds exactly nx members (selection sampling); the index guards keep
// the writes inside the map whatever the words hold.
__global__ void __launch_bounds__(256) k_rowmap(const uint32_t* __restrict__ words, int64_t count,
                                                int64_t n, int64_t nx,
                                                int32_t* __restrict__ rowmap) {
  __shared__ int32_t scan[256];
  const int64_t b = blockIdx.x;
  int32_t* map = rowmap + b * n;
  const int tid = threadIdx.x;
  if (b >= count) {
    for (int64_t t = tid; t < n; t += 256) map[t] = (int32_t)t;
    return;
  }
  const int64_t W = (n + 31) / 32;
  const uint32_t* z = words + b * W;
  int64_t base = 0;  // x* members in the words before the current run of 256
  for (int64_t w0 = 0; w0 < W; w0 += 256) {
    const int64_t w = w0 + tid;
    uint32_t word = w < W ? z[w] : 0u;
    if (w == W - 1 && (n & 31)) word &= (1u << (n & 31)) - 1u;
    const int c = __popc(word);
    scan[tid] = c;
    __syncthreads();
    for (int off = 1; off < 256; off <<= 1) {  // inclusive scan of the member counts
      const int v = tid >= off ? scan[tid - off] : 0;
      __syncthreads();
      scan[tid] += v;
      __syncthreads();
    }
    int64_t xr = base + scan[tid] - c;  // members before item 32 w
    const int64_t run = scan[255];
    __syncthreads();
    if (w < W) {
      for (int k = 0; k < 32; ++k) {
        const int64_t t = w * 32 + k;
        if (t >= n) break;
        if ((word >> k) & 1u) {
          if (xr < nx) map[xr] = (int32_t)t;
          ++xr;
        } else {
          const int64_t yr = t - xr;  // y* items before t
          if (yr < n - nx) map[nx + yr] = (int32_t)t;
        }
      }
    }
    base += run;
  }
}

// Flag words of m recomputations: the staging's non-finite flag and input maximum, the rest 0.
__global__ void k_sum_flags(const TestDesc* __restrict__ descs, int m,
                            const int32_t* __restrict__ staged) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= m) return;
  int32_t* f = descs[k].flags;
#pragma unroll
  for (int w = 0; w < FLAG_WORDS; ++w) f[w] = w == 0 || w == FLAG_XMAX ? staged[w] : 0;
}

// Statistic of each recomputed test (its observed statistic, eq. 1 / eq. 2) into the list
// of split statistics; the identity split's refined-pair count; non-finite input.
__global__ void k_collect(const TestDesc* __restrict__ descs, int m, int64_t c0, int64_t B,
                          double* __restrict__ stats, int32_t* __restrict__ flags) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= m) return;
  const TestDesc& d = descs[k];
  stats[c0 + k] = d.obs[3];
  if (d.flags[0]) atomicOr(&flags[0], 1);
  if (c0 + k == B) flags[1] = d.flags[1];
}

// Threshold (the identity split, stats[B]), exceedance count and p-value; copies the drawn
// splits' statistics to perm_out when given and the input was finite.
__global__ void __launch_bounds__(1024) k_count(const double* __restrict__ stats, int64_t B,
                                                const int32_t* __restrict__ flags,
                                                double* __restrict__ perm_out,
                                                DevResult* __restrict__ result) {
  __shared__ int64_t red[1024];
  const int tid = threadIdx.x;
  const double thr = stats[B];
  const bool bad = flags[0] != 0;
  int64_t c = 0;
  for (int64_t b = tid; b < B; b += 1024) {
    const double v = stats[b];
    c += v >= thr ? 1 : 0;
    if (perm_out && !bad) perm_out[b] = v;
  }
  red[tid] = c;
  __syncthreads();
  for (int s = 512; s > 0; s >>= 1) {
    if (tid < s) red[tid] += red[tid + s];
    __syncthreads();
  }
  if (tid == 0) {
    DevResult r;
    r.statistic = thr;
    r.threshold = thr;
    r.count_ge = red[0];
    r.B = B;
    r.p_value = (1.0 + (double)red[0]) / (1.0 + (double)B);
    r.n_refined = flags[1];
    r.status = bad ? 2 : 0;
    r.pad = 0;
    if (bad) {
      r.statistic = __builtin_nan("");
      r.threshold = __builtin_nan("");
      r.p_value = __builtin_nan("");
    }
    *result = r;
  }
}

// ------------------------------------------------------------ pre-computation test
// The stored upper tiles of the pooled Gram are the pooled matrix D_WW (each unordered
// pair once; diagonal tiles in full).  For split z (bit 1 = x*), with row sums over the
// tile's x* columns s_x and y* columns s_y, the three block sums of the split are
//   off-diagonal tile: row in x*: W_xx += 2 s_x, W_xy += s_y;  row in y*: W_xy += s_x,
//                      W_yy += 2 s_y   (each entry stands for (a, b) and (b, a));
//   diagonal tile:     row in x*: W_xx += s_x, W_xy += s_y;    row in y*: W_yy += s_y
//                      (the tile holds both orders; x*-y* pairs are taken once).
// With the dense pooled matrix (Alg. 5 as printed: every tile of the nt x nt grid, D_YX
// included) every tile holds both orders of its pairs and takes the diagonal-tile rule: the
// X*X*, Y*Y* and X*Y* sub-blocks are read entry by entry and the Y*X* entries are skipped.
// Padding entries are 0.  One workgroup per (tile, 32-row strip, 64 splits), 16 splits per wave:
// every entry of the strip is multiplied by each split's column bit as 0.0 or 1.0, which adds the
// entry or leaves the sum as it is, and added in FP64 -- on v_mfma_f64_16x16x4f64, 2 row blocks of 16 x 16; s_y
// is the row's total less s_x.  No centring and no quadratic form: this
// is the per-split extraction of Alg. 5.  The lanes read their entries straight from the
// stored tile (four adjacent columns each, FP32 entries converted) and the waves of a workgroup
// meet in the L1, the workgroups of a strip in one XCD's L2.  Bound by the FP64 MFMA rate; 211 us
// on the vector ALU (one FMA per entry and split, one wave per SIMD) -> 28 us for 1000 + 1000
// rows and 201 splits (34 with 64 splits per wave, where two rounds of the chip were one and a
// bit).
typedef double f64x4 __attribute__((ext_vector_type(4)));

// four adjacent entries
__device__ inline void load4(const float* p, double (&v)[4]) {
  const float4 x = *(const float4*)p;
  v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
}
__device__ inline void load4(const double* p, double (&v)[4]) {
  const double2 x = *(const double2*)p, y = *(const double2*)(p + 2);
  v[0] = x.x; v[1] = x.y; v[2] = y.x; v[3] = y.y;
}

template <typename T>
__global__ void __launch_bounds__(256) k_precomp(const TestDesc* __restrict__ descs,
                                                 double* __restrict__ part, int64_t sg,
                                                 int64_t first) {
  const TestDesc& d = descs[0];
  const int64_t id = xcd_grouped(blockIdx.x, gridDim.x);
  const int64_t g = id % sg;           // group of 64 split columns
  const int64_t u = first + id / sg;  // strip u: tile u / PC_STRIPS, rows 32 (u % PC_STRIPS) ..
  const int t = (int)(u / PC_STRIPS), h = (int)(u % PC_STRIPS);
  int i, j;
  if (d.dense) {
    i = t / d.nt;
    j = t % d.nt;
  } else {
    tile_coords(t, d.nt, &i, &j);
  }
  const int lane = threadIdx.x & 63, cl = lane & 15, kq = lane >> 4;
  const int64_t BP = d.B_pad, col = g * 64 + (threadIdx.x >> 6) * 16 + cl;  // Z columns past B are 0
  // the strip's rows cl and 16 + cl, columns 4 kq .. + 3 of every 16
  const T* src = (const T*)d.D + (int64_t)t * TILE * TILE + (h * PC_ROWS + cl) * TILE + 4 * kq;
  const uint32_t* Zj = d.Z + (int64_t)j * TILE_WORDS * BP + col;
  f64x4 acc[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
  // steps of 32 columns (one membership word), the next step's entries loaded ahead
  double a[2][2][4], an[2][2][4];
  uint32_t z, zn;
  auto load = [&](int s, double (&x)[2][2][4], uint32_t& y) {
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
      for (int q = 0; q < 2; ++q) load4(src + rb * 16 * TILE + 32 * s + 16 * q, x[rb][q]);
    y = Zj[(int64_t)s * BP];
  };
  // a step's products in a chain of their own, which loses less to a large entry than one over
  // the tile's 128 columns would; the chains of the four steps are added in pairs
  auto multiply = [&](const double (&x)[2][2][4], uint32_t y, f64x4 (&sum)[2]) {
    sum[0] = sum[1] = f64x4{0.0, 0.0, 0.0, 0.0};
    // column 16 q + 4 kq + e of the step: bit 16 q + e of the shifted word
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int bit = __builtin_amdgcn_sbfe((int)(y >> (4 * kq)), 16 * q + e, 1);
        const double b = __hiloint2double(bit & 0x3FF00000, 0);
#pragma unroll
        for (int rb = 0; rb < 2; ++rb)
          sum[rb] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[rb][q][e], b, sum[rb], 0, 0, 0);
      }
  };
  load(0, a, z);
#pragma unroll 1
  for (int s = 0; s < TILE_WORDS; s += 2) {
    f64x4 u[2], v[2];
    load(s + 1, an, zn);
    multiply(a, z, u);
    if (s + 2 < TILE_WORDS) load(s + 2, a, z);
    multiply(an, zn, v);
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) acc[rb] += u[rb] + v[rb];
  }
  // element e of an accumulator is row 16 rb + kq + 4 e of the strip, whose total the Gram left
  const double* ts = d.tsum + (int64_t)t * d.tsum_stride + h * PC_ROWS + kq;
  double tot[2][4];
#pragma unroll
  for (int rb = 0; rb < 2; ++rb)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const double* p = ts + 16 * rb + 4 * e;
      tot[rb][e] = sizeof(T) == 8 ? p[0] + p[TILE] : p[0];
    }
  // a tile holding both orders of its pairs: a diagonal tile, or any tile of the dense matrix
  const bool both_orders = d.dense || i == j;
  const uint32_t zr = d.Z[(int64_t)(i * TILE_WORDS + h) * BP + col] >> kq;
  double wxx = 0.0, wyy = 0.0, wxy = 0.0;
#pragma unroll
  for (int rb = 0; rb < 2; ++rb)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const double sx = acc[rb][e], sy = tot[rb][e] - sx;
      const bool member = (zr >> (16 * rb + 4 * e)) & 1u;
      wxx += member ? sx : 0.0;
      wyy += member ? 0.0 : sy;
      wxy += member ? sy : both_orders ? 0.0 : sx;
    }
  const double scale = both_orders ? 1.0 : 2.0;
  double w[3] = {scale * wxx, scale * wyy, wxy};
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    w[k] += __shfl_xor(w[k], 16, 64);
    w[k] += __shfl_xor(w[k], 32, 64);
  }
  if (kq == 0 && col <= d.B) {
#pragma unroll
    for (int k = 0; k < 3; ++k) part[(u * 3 + k) * BP + col] = w[k];
  }
}

struct Csum2 {  // Neumaier-compensated sum
  double s = 0.0, c = 0.0;
  __device__ void add(double x) {
    const double t = s + x;
    if (fabs(s) >= fabs(x)) c += (s - t) + x;
    else c += (x - t) + s;
    s = t;
  }
  __device__ double value() const { return s + c; }
};

// Statistics of 16 split columns per workgroup: 64 groups of lanes each take every 64th strip
// (compensated sums, the loads of two strips together), then the first adds the group sums in
// order (64 columns in 16 groups left 34 strips in turn to each lane of 4 workgroups: 16 us
// for 136 tiles, 10 us now).
constexpr int PCS_COLS = 16, PCS_GROUPS = 64;
__global__ void __launch_bounds__(PCS_COLS * PCS_GROUPS) k_precomp_stat(
    const TestDesc* __restrict__ descs, const double* __restrict__ part, int64_t nstrips,
    double* __restrict__ stats) {
  __shared__ double red[3][PCS_GROUPS][PCS_COLS];
  const TestDesc& d = descs[0];
  const int c = threadIdx.x % PCS_COLS, g = threadIdx.x / PCS_COLS;
  const int64_t s = (int64_t)blockIdx.x * PCS_COLS + c, BP = d.B_pad;  // s < B_pad
  Csum2 acc[3];
#pragma unroll 2
  for (int64_t u = g; u < nstrips; u += PCS_GROUPS) {
    double x[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) x[k] = part[(u * 3 + k) * BP + s];
#pragma unroll
    for (int k = 0; k < 3; ++k) acc[k].add(x[k]);
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) red[k][g][c] = acc[k].value();
  __syncthreads();
  if (g != 0 || s > d.B) return;
  Csum2 w[3];
#pragma unroll 4
  for (int q = 0; q < PCS_GROUPS; ++q)
#pragma unroll
    for (int k = 0; k < 3; ++k) w[k].add(red[k][q][c]);
  const double nx = d.nx, ny = d.ny;
  const double txx = w[0].value() / (nx * nx), tyy = w[1].value() / (ny * ny);
  const double txy = 2.0 * w[2].value() / (nx * ny);
  stats[s] = d.kind == KIND_ED ? (txy - txx) - tyy : (txx + tyy) - txy;
}

// ------------------------------------------------------------------- launchers
void launch_rowmap(const uint32_t* words, int64_t count, int64_t maps, int64_t n, int64_t nx,
                   int32_t* rowmap, hipStream_t st) {
  if (maps > 0)
    hipLaunchKernelGGL(k_rowmap, dim3((unsigned)maps), dim3(256), 0, st, words, count, n, nx,
                       rowmap);
}
void launch_sum_flags(const TestDesc* d, int m, const int32_t* staged, hipStream_t st) {
  if (m > 0)
    hipLaunchKernelGGL(k_sum_flags, dim3((unsigned)((m + 255) / 256)), dim3(256), 0, st, d, m,
                       staged);
}
void launch_collect(const TestDesc* d, int m, int64_t c0, int64_t B, double* stats,
                    int32_t* flags, hipStream_t st) {
  if (m > 0)
    hipLaunchKernelGGL(k_collect, dim3((unsigned)((m + 255) / 256)), dim3(256), 0, st, d, m, c0, B,
                       stats, flags);
}
void launch_count(const double* stats, int64_t B, const int32_t* flags, double* perm_out,
                  DevResult* result, hipStream_t st) {
  hipLaunchKernelGGL(k_count, dim3(1), dim3(1024), 0, st, stats, B, flags, perm_out, result);
}
// Strip sums of every split column: ntiles * PC_STRIPS strips x ceil((B + 1) / 64) groups.
void launch_precomp(bool f64, const TestDesc* d, int64_t ntiles, int64_t B, double* part,
                    hipStream_t st) {
  const int64_t sg = (B + 1 + 63) / 64, strips = ntiles * PC_STRIPS;
  // several dispatches of at most 2^23 workgroups
  const int64_t most = ((int64_t)1 << 23) / sg > 0 ? ((int64_t)1 << 23) / sg : 1;
  for (int64_t first = 0; first < strips; first += most) {
    const dim3 grid((unsigned)(std::min(most, strips - first) * sg));
    if (f64) hipLaunchKernelGGL(k_precomp<double>, grid, dim3(256), 0, st, d, part, sg, first);
    else hipLaunchKernelGGL(k_precomp<float>, grid, dim3(256), 0, st, d, part, sg, first);
  }
}
void launch_precomp_stat(const TestDesc* d, int64_t ntiles, int64_t B, const double* part,
                         double* stats, hipStream_t st) {
  hipLaunchKernelGGL(k_precomp_stat, dim3((unsigned)((B + PCS_COLS) / PCS_COLS)),
                     dim3(PCS_COLS * PCS_GROUPS), 0, st, d, part, ntiles * PC_STRIPS, stats);
}

}  // namespace et
