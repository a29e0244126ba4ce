// HSIC independence permutation test (the extension proposed in the paper's discussion):
// paired samples (x_i, y_i), i < n; Gaussian kernel matrices K of x and L of y are
// computed once (the staging and Gram kernels of the two-sample test, one "sample" each);
// each permutation pi of the y sample then costs one pass over the n^2 entries:
//   Kt = K - diag(K), Lt = L - diag(L), r = Kt 1, s = Lt 1,
//   T1(pi) = sum_{i,j} Kt[i][j] Lt[pi_i][pi_j],  T3(pi) = sum_i r_i s_{pi_i},
//   T2 = (1^T Kt 1)(1^T Lt 1),
//   HSIC(pi) = [T1 + T2 / ((n-1)(n-2)) - 2 T3 / (n-2)] / (n (n-3))
// (the unbiased estimator of Song et al. 2012).  Unlike the two-sample statistics, T1 is
// not a quadratic form in a 0/1 vector, so no contraction shortens it: each permutation
// gathers n^2 entries of Lt, the cost the discussion anticipates.
#include "common.h"

#include <type_traits>

namespace et {

// ------------------------------------------------------------------ permutations
// Permutation b of 0..n-1: items ordered by a 64-bit Philox4x32-10 key, key (seed_lo,
// seed_hi), counter (t/2, b_lo, b_hi, 1) (even t: words 0, 1; odd t: words 2, 3; low word
// first), ties by index.  One workgroup per permutation: a bitonic sort of (key, item) in
// LDS over the next power of two (padding keys all ones, padding items >= n, so they sort
// after every real item).  perms[q][i] = the item placed at position i, for b = b0 + q with
// q < count; slots count .. total - 1 hold the identity.  The test itself takes 16-bit tables
// of row stride ld instead (perms null): p16[q][i] as above (0 past n) and the inverse
// inv16[q][item] = position (0xFFFF past n).
__device__ inline uint64_t perm_key(uint32_t k0, uint32_t k1, uint32_t b_lo, uint32_t b_hi,
                                    uint32_t t) {
  const uint4 r = philox4x32_10(make_uint4(t >> 1, b_lo, b_hi, 1u), k0, k1);
  return (t & 1u) ? ((uint64_t)r.w << 32) | r.z : ((uint64_t)r.y << 32) | r.x;
}

__global__ void __launch_bounds__(1024) k_permgen(int64_t n, uint64_t seed, int64_t b0,
                                                  int64_t count, int32_t* __restrict__ perms,
                                                  uint16_t* __restrict__ p16,
                                                  uint16_t* __restrict__ inv16, int64_t ld) {
  __shared__ uint64_t key[HSIC_NMAX];
  __shared__ int32_t item[HSIC_NMAX];
  const int64_t q = blockIdx.x;
  const int tid = threadIdx.x;
  auto put = [&](int64_t t, int32_t it) {
    if (perms) perms[q * n + t] = it;
    else {
      p16[q * ld + t] = (uint16_t)it;
      inv16[q * ld + it] = (uint16_t)t;
    }
  };
  if (!perms)
    for (int64_t t = n + tid; t < ld; t += 1024) {
      p16[q * ld + t] = 0;
      inv16[q * ld + t] = 0xFFFFu;
    }
  if (q >= count) {
    for (int64_t t = tid; t < n; t += 1024) put(t, (int32_t)t);
    return;
  }
  const uint64_t b = (uint64_t)(b0 + q);
  const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
  int n2 = 1;
  while (n2 < n) n2 <<= 1;
  for (int t = tid; t < n2; t += 1024) {
    key[t] = t < n ? perm_key(k0, k1, (uint32_t)b, (uint32_t)(b >> 32), (uint32_t)t) : ~0ull;
    item[t] = t;
  }
  __syncthreads();
  for (int k = 2; k <= n2; k <<= 1) {
    for (int j = k >> 1; j > 0; j >>= 1) {
      for (int t = tid; t < n2; t += 1024) {
        const int l = t ^ j;
        if (l > t) {
          const bool ascending = (t & k) == 0;
          const uint64_t kt = key[t], kl = key[l];
          const int32_t it = item[t], il = item[l];
          const bool greater = kt > kl || (kt == kl && it > il);
          if (greater == ascending) {
            key[t] = kl;
            key[l] = kt;
            item[t] = il;
            item[l] = it;
          }
        }
      }
      __syncthreads();
    }
  }
  for (int64_t t = tid; t < n; t += 1024) put(t, item[t]);
}

// ------------------------------------------------------------------ kernel matrix of x
// T1(pi) = sum over ordered pairs i != j of Kt[i][j] Lt[pi_i][pi_j].  Both matrices are
// symmetric up to the last bit of the entries inside a diagonal tile, where the Gram forms
// (i, j) and (j, i) apart.  With S[a][b] = Lt[a][b] + Lt[b][a], every unordered pair is
// therefore taken once, as Kt[i][j] S[pi_i][pi_j], or, for i and j in one tile, twice as half
// of that (which differs by a product of two such last bits only).  The dense matrix written
// here holds those weights of Kt: a pair of different tiles belongs to the row i from which j
// lies at most n / 2 ahead, cyclically (at exactly n / 2: to the smaller of the two), so that
// every range of columns carries the same work; its other entry is 0.  FP32 entries are
// scaled by 2^127 (see HT_SCALE).  Row-major, n rows of stride ld; columns from n on are 0.
template <typename T>
__device__ inline T hsic_weight(T v, int64_t i, int64_t j, int64_t n) {
  int64_t dl = j - i;
  dl += dl < 0 ? n : 0;
  T w;
  if (i / TILE == j / TILE) w = i == j ? (T)0 : (T)0.5;
  else w = 2 * dl < n || (2 * dl == n && j > i) ? (T)1 : (T)0;
  if (sizeof(T) == 4) w *= (T)0x1p127;
  return j < n ? v * w : (T)0;
}

// One workgroup per stored tile and 32-row strip, which it writes as it is and, off the
// diagonal, transposed through LDS.
template <typename T>
__global__ void __launch_bounds__(256) k_hsic_dense(const TestDesc* __restrict__ descs, int64_t n,
                                                    int64_t ld, T* __restrict__ kx) {
  __shared__ T strip[32][TILE + 1];
  const TestDesc& d = descs[0];
  const int t = (int)(blockIdx.x >> 2), s = (int)(blockIdx.x & 3);
  int i, j;
  tile_coords(t, d.nt, &i, &j);
  const T* src = (const T*)d.D + (int64_t)t * TILE * TILE + s * 32 * TILE;
  const int tid = threadIdx.x;
  const int64_t r0 = (int64_t)i * TILE + s * 32, c0 = (int64_t)j * TILE;
  T v[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) v[k] = src[tid + 256 * k];
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const int r = (tid + 256 * k) >> 7, c = tid & (TILE - 1);
    strip[r][c] = v[k];
    if (r0 + r < n) kx[(r0 + r) * ld + c0 + c] = hsic_weight(v[k], r0 + r, c0 + c, n);
  }
  if (j == d.nt - 1)  // the columns past the last tile
    for (int64_t c = c0 + TILE + (tid & 31); c < ld; c += 32)
      for (int r = tid >> 5; r < 32; r += 8)
        if (r0 + r < n) kx[(r0 + r) * ld + c] = (T)0;
  if (i == j) return;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const int c = (tid >> 5) + 8 * k, r = tid & 31;
    if (c0 + c < n) kx[(c0 + c) * ld + r0 + r] = hsic_weight(strip[r][c], c0 + c, r0 + r, n);
  }
}

// Row sums r = Kt 1 and s = Lt 1 in FP64, one workgroup per tile row and matrix
// (blockIdx.y): the sums the Gram left per stored tile and, in the diagonal tile, the row's
// entries without the diagonal one (which would swallow the others where they are small).
// Eight threads per row, combined by a fixed butterfly.
template <typename T>
__global__ void __launch_bounds__(1024) k_hsic_rows(const TestDesc* __restrict__ descs, int64_t n,
                                                    double* __restrict__ rx,
                                                    double* __restrict__ ry) {
  const TestDesc& d = descs[blockIdx.y];
  const int i = blockIdx.x, r = threadIdx.x >> 3, q = threadIdx.x & 7;
  const T* row = (const T*)d.D + tile_index(i, i, d.nt) * TILE * TILE + r * TILE + q * 16;
  T v[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) v[e] = row[e];
  double s = 0.0;
#pragma unroll
  for (int e = 0; e < 16; ++e) s += q * 16 + e == r ? 0.0 : (double)v[e];
#pragma unroll 2
  for (int j = q; j < d.nt; j += 8) {
    if (j == i) continue;
    const double* t = d.tsum + tile_index(min(i, j), max(i, j), d.nt) * d.tsum_stride + r;
    if (sizeof(T) == 8)
      s += j > i ? t[0] + t[TILE]
                 : (t[2 * TILE] + t[3 * TILE]) + (t[4 * TILE] + t[5 * TILE]);
    else
      s += j > i ? t[0] : t[TILE] + t[2 * TILE];
  }
#pragma unroll
  for (int m = 1; m < 8; m <<= 1) s += __shfl_xor(s, m, 64);
  const int64_t pos = (int64_t)i * TILE + r;
  if (q == 0 && pos < n) (blockIdx.y == 0 ? rx : ry)[pos] = s;
}

struct Hsum {  // Neumaier-compensated sum
  double s = 0.0, c = 0.0;
  __device__ void add(double x) {
    const double t = s + x;
    if (fabs(s) >= fabs(x)) c += (s - t) + x;
    else c += (x - t) + s;
    s = t;
  }
  __device__ double value() const { return s + c; }
};

// Totals 1^T Kt 1 and 1^T Lt 1 (hs[0], hs[1]; one workgroup each), and the two staging flags
// merged for the count (flags[0]: non-finite input in x or y; flags[1]: refined pairs of both
// Grams).
__global__ void __launch_bounds__(1024) k_hsic_sums(const TestDesc* __restrict__ descs, int64_t n,
                                                    const double* __restrict__ rx,
                                                    const double* __restrict__ ry,
                                                    double* __restrict__ hs,
                                                    int32_t* __restrict__ flags) {
  __shared__ double red[2][1024];
  const int tid = threadIdx.x;
  const double* src = blockIdx.x == 0 ? rx : ry;
  double v[HSIC_NMAX / 1024];
#pragma unroll
  for (int k = 0; k < HSIC_NMAX / 1024; ++k) v[k] = tid + 1024 * k < n ? src[tid + 1024 * k] : 0.0;
  Hsum a;
#pragma unroll
  for (int k = 0; k < HSIC_NMAX / 1024; ++k) a.add(v[k]);
  red[0][tid] = a.s;
  red[1][tid] = a.c;
  for (int st = 512; st > 0; st >>= 1) {  // compensated pairwise combination, fixed tree
    __syncthreads();
    if (tid < st) {
      a.c += red[1][tid + st];
      a.add(red[0][tid + st]);
      red[0][tid] = a.s;
      red[1][tid] = a.c;
    }
  }
  if (tid == 0) hs[blockIdx.x] = a.value();
  if (tid == 0 && blockIdx.x == 0) {
    flags[0] = (descs[0].flags[0] | descs[1].flags[0]) ? 1 : 0;
    flags[1] = descs[0].flags[1] + descs[1].flags[1];
  }
}

// ------------------------------------------------------------------ permutations' terms
// A workgroup holds G rows l of S in LDS and one slice of 256 columns j.  A wave takes one
// permutation at a time: its lanes hold pi_j of four columns each, and for every staged row l
// the weighted row i = pi^-1(l) of Kt is read along the slice (coalesced, one permutation
// ahead) while the lanes gather S[l][pi_j] from LDS.  Rows that own no pair of the slice are
// skipped.  So each row of S is staged once per slice instead of once per permutation, and
// half of the pairs' entries are never touched.  The products of two FP32 entries are exact
// in FP64; a lane adds CH of a row's four, then adds such chains, and the wave its lanes, with
// compensation (the three terms of the estimator cancel to a small fraction of their size), and
// so are the waves' sums (part[b][slice][group]).  Bound by the vector ALU in the FP32 form (76%
// busy, the gathers' random LDS banks 58%).
//
// FP32 form: S has one bit more than an FP32 value and no sign, so it is staged as 8 exponent
// and 24 mantissa bits: bits 28..59 of the FP64 value S 2^-896, which two shifts restore.
// Kt carries 2^127.  A product is then an integer times 2^-1068 (entries are integers times
// 2^-149, halves of them times 2^-150), which FP64 holds exactly from its normal range, products
// of 2^-253, down through its subnormals (multiples of 2^-1074); the sums are scaled back by
// 2^769.
//
// Units are slice-major and every XCD takes a contiguous run of them: the Kt entries of one
// slice (2 MB at n = 2000) stay in its L2 across all permutations (95% of the reads hit).
//
// Measured at n = 2000 and 201 permutations: 1007 us with one workgroup per permutation and
// 8 rows (a row of Lt staged for each of them, every entry read), 416 us in this form without
// the reads one permutation ahead and with the pairs' ownership tested per entry, 201 us with it
// tested row by row on the scalar unit, 155 us with them chosen over the lanes but every sum of a
// wave by plain additions (vector ALU 60% busy, LDS 65%), 179 us now.  Whole tests, plain / now:
// that one 286 / 303 us, n = 4096 1000 / 1111 (1147 with the lanes' sums by ds_bpermute); FP64
// form 1780 / 1795.  Four rows interleaved, so that one 16-byte read gathers them all: 314 us, 54
// LDS cycles per read.
constexpr int HT_THREADS = 512;
constexpr int HT_COLS = 256;   // columns per slice
constexpr int HT_BATCH = 4;    // permutations per wave whose sums are combined together
constexpr int HT_SCALE = 769;  // FP32 form: the sums' exponent offset, 896 - 127
template <typename T>
constexpr int HT_G = 32 / sizeof(T);  // rows of S per workgroup

// four consecutive entries
__device__ inline void load4(const float* p, float (&v)[4]) {
  const float4 x = *(const float4*)p;
  v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
}
__device__ inline void load4(const double* p, double (&v)[4]) {
  const double2 x = *(const double2*)p, y = *(const double2*)(p + 2);
  v[0] = x.x; v[1] = x.y; v[2] = y.x; v[3] = y.y;
}

// a + b as it is staged (exact: at most 25 significant bits, or an FP64 sum), and its value
__device__ inline uint32_t stage_sum(float a, float b) {
  const double s = ((double)a + (double)b) * 0x1p-896;
  return (uint32_t)(__double_as_longlong(s) >> 28);
}
__device__ inline double stage_sum(double a, double b) { return a + b; }
__device__ inline double staged(uint32_t u) { return __hiloint2double((int)(u >> 4), (int)(u << 28)); }
__device__ inline double staged(double v) { return v; }

// A sum and the roundings it has left behind (the error-free sum of two numbers, whatever their
// order).
struct Pair {
  double s = 0.0, c = 0.0;
  __device__ void add(double x) {
    const double t = s + x, b = t - s;
    c += (s - (t - b)) + (x - b);
    s = t;
  }
  __device__ void add(const Pair& x) {
    c += x.c;
    add(x.s);
  }
};
// Two sums over the lanes become one: lanes 0 .. 31 (row 16 even) hold a's, the others b's, each
// with the other half's (the other row's) share added.
template <int LANES>
__device__ inline Pair join(const Pair& a, const Pair& b) {
  auto exchange = [](double& x, double& y) {
    const uint64_t u = __builtin_bit_cast(uint64_t, x), v = __builtin_bit_cast(uint64_t, y);
    uint32_t p[2] = {(uint32_t)u, (uint32_t)(u >> 32)}, q[2] = {(uint32_t)v, (uint32_t)(v >> 32)};
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const auto r = LANES == 32 ? __builtin_amdgcn_permlane32_swap(p[k], q[k], false, false)
                                 : __builtin_amdgcn_permlane16_swap(p[k], q[k], false, false);
      p[k] = r[0];
      q[k] = r[1];
    }
    x = __builtin_bit_cast(double, (uint64_t)p[1] << 32 | p[0]);
    y = __builtin_bit_cast(double, (uint64_t)q[1] << 32 | q[0]);
  };
  Pair x = a, y = b;
  exchange(x.s, y.s);
  exchange(x.c, y.c);
  x.add(y);
  return x;
}
// the value of the lane N places on, cyclically within 16
template <int N>
__device__ inline double rotated(double x) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)u, 0x120 + N, 0xf, 0xf, true),
                 hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), 0x120 + N, 0xf, 0xf, true);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
template <int N>
__device__ inline void add_rotated(Pair& a) {
  Pair x;
  x.s = rotated<N>(a.s);
  x.c = rotated<N>(a.c);
  a.add(x);
}
// NC: columns of a staged row (a power of two, at least the tiles' columns).  CH: products of
// a row that a lane adds before a compensated step.
template <typename T, int NC, int CH>
__global__ void __launch_bounds__(HT_THREADS) __attribute__((amdgpu_waves_per_eu(4)))
k_hsic_terms(const TestDesc* __restrict__ descs, const T* __restrict__ kx, int n, int ld,
             const uint16_t* __restrict__ p16, const uint16_t* __restrict__ inv16, int nperm,
             int nsl, int ngrp, int nps, double* __restrict__ part) {
  typedef decltype(stage_sum(T(), T())) ST;
  constexpr int G = HT_G<T>;
  __shared__ ST lt[G][NC];
  // unit (slice, row group, permutation range): contiguous runs per XCD
  const int64_t units = (int64_t)nsl * ngrp * nps, run = (units + NUM_XCD - 1) / NUM_XCD;
  const int64_t u = (int64_t)(blockIdx.x % NUM_XCD) * run + blockIdx.x / NUM_XCD;
  if (u >= units) return;
  const int sl = (int)(u / ((int64_t)ngrp * nps));
  const int rem = (int)(u % ((int64_t)ngrp * nps));
  const int grp = rem / nps, ps = rem % nps;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l0 = grp * G;
  {  // rows l0 .. l0 + G - 1 of S from the stored upper tiles: row pieces of tile (I, J),
     // J > I; below the diagonal the same entries are columns of tile (J, I); both inside the
     // diagonal tile (whose diagonal meets weights of 0 only)
    const TestDesc& d = descs[1];
    const int I = l0 / TILE, r = l0 % TILE;
    const T* D = (const T*)d.D;
    for (int m = tid; m < d.nt * TILE; m += HT_THREADS) {
      const int J = m / TILE, c = m % TILE;
      T v[G], x[G];
      if (J >= I) {
        const T* src = D + tile_index(I, J, d.nt) * TILE * TILE + r * TILE + c;
#pragma unroll
        for (int g = 0; g < G; ++g) v[g] = src[g * TILE];
      }
      if (J <= I) {
        const T* src = D + tile_index(J, I, d.nt) * TILE * TILE + c * TILE + r;
#pragma unroll
        for (int g = 0; g < G; g += 4) {
          T y[4];
          load4(src + g, y);
#pragma unroll
          for (int e = 0; e < 4; ++e) x[g + e] = y[e];
        }
      }
#pragma unroll
      for (int g = 0; g < G; ++g)
        lt[g][m] = stage_sum(J >= I ? v[g] : x[g], J <= I ? x[g] : v[g]);
    }
  }
  __syncthreads();
  const int c0 = sl * HT_COLS, j0 = c0 + 4 * lane;
  // this unit's permutations [b0, b1); wave w takes batches of HT_BATCH
  const int per = ((nperm + nps - 1) / nps + HT_BATCH - 1) / HT_BATCH * HT_BATCH;
  const int b0 = ps * per, b1 = min(nperm, b0 + per);
  constexpr int STEP = HT_BATCH * (HT_THREADS / 64);
  struct Tables {
    ushort4 pj[HT_BATCH];
    uint16_t i;  // lane q G + g: the row of Kt that meets row l0 + g of S in permutation q
  };
  const int tq = lane / G % HT_BATCH, tg = lane % G;
  auto tables = [&](int bb, Tables& t) {
#pragma unroll
    for (int q = 0; q < HT_BATCH; ++q)
      t.pj[q] = *(const ushort4*)(p16 + (int64_t)min(bb + q, nperm - 1) * ld + j0);
    t.i = inv16[(int64_t)min(bb + tq, nperm - 1) * ld + l0 + tg];
  };
  // the batch's rows of Kt, all in one step over the lanes: bit q G + g of the result tells that
  // the row owns a pair of the slice, off its place; the others' loads go to row 0 (always the
  // same line).  (Row by row on the scalar unit this was 14 instructions each, two thirds of the
  // scalar unit's time.)
  auto choose = [&](const Tables& t, uint32_t& off) {
    const int i = t.i;
    int d0 = c0 - i;  // cyclic distance of the slice's first column
    d0 += d0 < 0 ? n : 0;
    const bool a = i < n && ((i / HT_COLS) == sl || 2 * d0 <= n);
    off = (a ? (uint32_t)i : 0u) * (uint32_t)(ld * sizeof(T));
    return (uint32_t)__ballot(a);
  };
  auto rows = [&](uint32_t off, int q, T (&kv)[G][4]) {
#pragma unroll
    for (int g = 0; g < G; ++g)
      load4((const T*)((const char*)kx + (uint32_t)__builtin_amdgcn_readlane(off, q * G + g)) + j0, kv[g]);
  };
  auto terms = [&](const Tables& t, int q, uint32_t all, const T (&kv)[G][4]) {
    const uint32_t on = all >> (q * G);
    const int pk[4] = {t.pj[q].x, t.pj[q].y, t.pj[q].z, t.pj[q].w};
    Pair a;
#pragma unroll
    for (int g = 0; g < G; ++g)
      if (on >> g & 1u) {
        double x = 0.0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          x = fma((double)kv[g][e], staged(lt[g][pk[e]]), x);
          if ((e + 1) % CH == 0) {
            a.add(x);
            x = 0.0;
          }
        }
      }
    return a;
  };
  Tables t, tn;
  T ka[G][4], kb[G][4];
  uint32_t off = 0, on = 0;
  int bb = b0 + w * HT_BATCH;
  if (bb < b1) {
    tables(bb, t);
    on = choose(t, off);
    rows(off, 0, ka);
  }
  static_assert(HT_BATCH == 4 && HT_BATCH * G <= 32, "the batch is written out, its rows are bits");
  for (; bb < b1; bb += STEP) {
    Pair acc[HT_BATCH];
    tables(min(bb + STEP, nperm - 1), tn);
    rows(off, 1, kb);
    acc[0] = terms(t, 0, on, ka);
    rows(off, 2, ka);
    acc[1] = terms(t, 1, on, kb);
    rows(off, 3, kb);
    acc[2] = terms(t, 2, on, ka);
    const uint32_t cur = on;
    on = choose(tn, off);
    rows(off, 0, ka);
    acc[3] = terms(t, 3, cur, kb);
    t = tn;
    // sums over the lanes, the four permutations together: lanes 16 k .. + 15 end with
    // permutation (k >> 1) + 2 (k & 1)
    const bool hi5 = lane & 32, hi4 = lane & 16;
    Pair sum = join<16>(join<32>(acc[0], acc[1]), join<32>(acc[2], acc[3]));
    add_rotated<8>(sum);
    add_rotated<4>(sum);
    add_rotated<2>(sum);
    add_rotated<1>(sum);
    double x = sum.s + sum.c;
    if (sizeof(T) == 4) x = ldexp(x, HT_SCALE);
    const int b = bb + (hi5 ? 1 : 0) + (hi4 ? 2 : 0);
    if ((lane & 15) == 0 && b < b1) part[((int64_t)b * nsl + sl) * ngrp + grp] = x;
  }
}

// HSIC of one permutation per workgroup: T1 from its partial sums, T3 = sum_i r_i s_{pi_i},
// both with compensation in a fixed order.
__global__ void __launch_bounds__(256) k_hsic_stat(const double* __restrict__ part, int64_t nparts,
                                                   int64_t n, int64_t ld,
                                                   const uint16_t* __restrict__ p16,
                                                   const double* __restrict__ rx,
                                                   const double* __restrict__ ry,
                                                   const double* __restrict__ hs,
                                                   double* __restrict__ stats) {
  __shared__ double red[4][256];
  const int64_t b = blockIdx.x;
  const int tid = threadIdx.x;
  Hsum t1, t3;
  const double* p = part + b * nparts;
#pragma unroll 8
  for (int64_t k = tid; k < nparts; k += 256) t1.add(p[k]);
#pragma unroll 4
  for (int64_t i = tid; i < n; i += 256) t3.add(rx[i] * ry[p16[b * ld + i]]);
  red[0][tid] = t1.s;
  red[1][tid] = t1.c;
  red[2][tid] = t3.s;
  red[3][tid] = t3.c;
  for (int st = 128; st > 0; st >>= 1) {
    __syncthreads();
    if (tid < st) {
      t1.c += red[1][tid + st];
      t1.add(red[0][tid + st]);
      t3.c += red[3][tid + st];
      t3.add(red[2][tid + st]);
      red[0][tid] = t1.s;
      red[1][tid] = t1.c;
      red[2][tid] = t3.s;
      red[3][tid] = t3.c;
    }
  }
  if (tid != 0) return;
  const double dn = (double)n;
  const double t2 = hs[0] * hs[1];
  stats[b] = (t1.value() + t2 / ((dn - 1.0) * (dn - 2.0)) - 2.0 * t3.value() / (dn - 2.0)) /
             (dn * (dn - 3.0));
}

// ------------------------------------------------------------------- launchers
void launch_permgen(int64_t n, uint64_t seed, int64_t b0, int64_t count, int64_t total,
                    int32_t* perms, hipStream_t st) {
  if (total > 0)
    hipLaunchKernelGGL(k_permgen, dim3((unsigned)total), dim3(1024), 0, st, n, seed, b0, count,
                       perms, (uint16_t*)nullptr, (uint16_t*)nullptr, (int64_t)0);
}
void launch_hsic_perms(int64_t n, int64_t ld, uint64_t seed, int64_t b0, int64_t count,
                       int64_t total, uint16_t* p16, uint16_t* inv16, hipStream_t st) {
  if (total > 0)
    hipLaunchKernelGGL(k_permgen, dim3((unsigned)total), dim3(1024), 0, st, n, seed, b0, count,
                       (int32_t*)nullptr, p16, inv16, ld);
}
void launch_hsic_prep(bool f64, const TestDesc* d, int64_t nt, int64_t n, int64_t ld, void* kx,
                      double* rx, double* ry, double* hs, int32_t* flags, hipStream_t st) {
  const dim3 g((unsigned)(nt * (nt + 1) / 2 * 4)), gr((unsigned)nt, 2);
  if (f64) {
    hipLaunchKernelGGL(k_hsic_dense<double>, g, dim3(256), 0, st, d, n, ld, (double*)kx);
    hipLaunchKernelGGL(k_hsic_rows<double>, gr, dim3(1024), 0, st, d, n, rx, ry);
  } else {
    hipLaunchKernelGGL(k_hsic_dense<float>, g, dim3(256), 0, st, d, n, ld, (float*)kx);
    hipLaunchKernelGGL(k_hsic_rows<float>, gr, dim3(1024), 0, st, d, n, rx, ry);
  }
  hipLaunchKernelGGL(k_hsic_sums, dim3(2), dim3(1024), 0, st, d, n, rx, ry, hs, flags);
}
int64_t hsic_parts(bool f64, int64_t n) {
  const int64_t g = f64 ? HT_G<double> : HT_G<float>;
  return (n + HT_COLS - 1) / HT_COLS * ((n + g - 1) / g);
}
void launch_hsic_terms(bool f64, const TestDesc* d, const void* kx, int64_t n, int64_t ld,
                       const uint16_t* p16, const uint16_t* inv16, int64_t nperm, double* part,
                       hipStream_t st) {
  const int64_t g = f64 ? HT_G<double> : HT_G<float>;
  const int nsl = (int)((n + HT_COLS - 1) / HT_COLS), ngrp = (int)((n + g - 1) / g);
  // permutation ranges per (slice, row group): enough units for three rounds of the chip's
  // 512 resident workgroups, but at least one batch for each of a workgroup's waves; each range
  // stages the rows again (n = 2000, plain additions: 2000 units in one range 155 us, 4000 in two 169)
  int nps = 1;
  while (nps < 64 && (int64_t)nsl * ngrp * nps < 1536 &&
         nperm >= 2 * nps * HT_BATCH * (HT_THREADS / 64))
    nps *= 2;
  const int64_t units = (int64_t)nsl * ngrp * nps;
  const dim3 grid((unsigned)((units + NUM_XCD - 1) / NUM_XCD * NUM_XCD));
  auto go = [&](auto* k, auto* x) {
    hipLaunchKernelGGL(k, grid, dim3(HT_THREADS), 0, st, d, x, (int)n, (int)ld, p16, inv16,
                       (int)nperm, nsl, ngrp, nps, part);
  };
  auto pick = [&](auto* x) {
    typedef std::remove_const_t<std::remove_pointer_t<decltype(x)>> T;
    // a chain of plain additions has at most n / 256 products, rounded up: as the number of
    // chains grows with n^2, its roundings stay below those of the partial sums
    if (n <= 256) go(k_hsic_terms<T, 512, 1>, x);
    else if (n <= 512) go(k_hsic_terms<T, 512, 2>, x);
    else if (n <= 768) go(k_hsic_terms<T, 1024, 2>, x);
    else if (n <= 1024) go(k_hsic_terms<T, 1024, 4>, x);
    else if (n <= 2048) go(k_hsic_terms<T, 2048, 4>, x);
    else go(k_hsic_terms<T, HSIC_NMAX, 4>, x);
  };
  if (f64) pick((const double*)kx);
  else pick((const float*)kx);
}
void launch_hsic_stat(const double* part, int64_t nparts, int64_t n, int64_t ld,
                      const uint16_t* p16, const double* rx, const double* ry, int64_t nperm,
                      const double* hs, double* stats, hipStream_t st) {
  hipLaunchKernelGGL(k_hsic_stat, dim3((unsigned)nperm), dim3(256), 0, st, part, nparts, n, ld,
                     p16, rx, ry, hs, stats);
}

}  // namespace et
