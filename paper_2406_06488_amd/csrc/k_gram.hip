// Block stage: the stored tiles (i <= j) of the pooled tile grid.  FP32 / BF16 forms: Gram tile G
// = W_i W_j^T on MFMA, a workgroup per half tile, tile or 2 x 2 tiles; epilogue d^2 = |w_a|^2 +
// |w_b|^2 - 2 g (clamped at 0), then D = sqrt(d^2) (energy distance, Alg. 3) or K = exp(-gamma
// d^2) (Gaussian kernel); pairs with d^2 < 1e-3 (|w_a|^2 + |w_b|^2) are recomputed as a direct FP32
// difference of the input rows.  The FP64 form evaluates Alg. 3 as written (sum of squared
// differences) on the vector ALU, a workgroup per 32 x 64 part of a tile.
//
// Every stored tile also yields FP64 row sums and column sums, from which the
// observed statistic (eq. 1 / eq. 2) and the double-centring constants follow.
#include "common.h"

namespace et {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

struct TileCtx {
  int t, i, j;
  int rows_i, rows_j;
  bool diag;
};

__device__ inline TileCtx tile_ctx(const TestDesc& d, int64_t local) {
  TileCtx c;
  c.t = (int)local;
  if (d.cross) {  // the rectangle x side by y side, row-major
    c.i = (int)(local / d.ty);
    c.j = d.tx + (int)(local % d.ty);
  } else if (d.dense) {  // the whole nt x nt grid, row-major
    c.i = (int)(local / d.nt);
    c.j = (int)(local % d.nt);
  } else {
    tile_coords(c.t, d.nt, &c.i, &c.j);
  }
  c.rows_i = tile_rows(d, c.i);
  c.rows_j = tile_rows(d, c.j);
  c.diag = c.i == c.j;
  return c;
}

// Input row (pooled, unpadded) of tile row r of pooled tile i.
__device__ inline const float* input_row_f32(const TestDesc& d, int i, int r) {
  const int64_t t = i < d.tx ? (int64_t)i * TILE + r : d.nx + (int64_t)(i - d.tx) * TILE + r;
  return pooled_row<float>(d, t);
}

// d^2 -> stored block value (distance, or Gaussian kernel with bandwidth 1 / gamma);
// padding rows/columns hold 0.
__device__ inline float block_value_f32(int kind, double gamma, const TileCtx& c, int r, int col,
                                        float d2) {
  if (r >= c.rows_i || col >= c.rows_j) return 0.0f;
  if (c.diag && r == col) return kind == KIND_ED ? 0.0f : 1.0f;
  d2 = fmaxf(d2, 0.0f);
  return kind == KIND_ED ? sqrtf(d2) : expf((float)(-gamma) * d2);
}

// The block outputs one epilogue pass writes: the test's own, or those of the MMD test it
// feeds (shared block stage).
struct BlockOut {
  int kind;
  int split;  // cross tests: y-side columns below `split` are x2, the rest y2; -1 otherwise
  double gamma;
  float* D;
  double* tsum;
  float* tmax;
};
// columns of y-side tile j that hold x2 rows (cross tests)
__device__ inline int cross_split(const TestDesc& d, int j) {
  const int s = d.cnx2 - (j - d.tx) * TILE;
  return s < 0 ? 0 : (s > TILE ? TILE : s);
}
__device__ inline BlockOut own_out(const TestDesc& d, const TileCtx& c) {
  const int64_t t = c.t;
  return BlockOut{d.kind, d.cross ? cross_split(d, c.j) : -1, d.gamma,
                  d.cross || !d.D ? nullptr : (float*)d.D + t * TILE * TILE,
                  d.tsum + t * d.tsum_stride, d.tmax + t * TMAX_PER_TILE};
}
__device__ inline BlockOut partner_out(const TestDesc& d, const TileCtx& c) {
  const int64_t t = c.t;
  return BlockOut{KIND_MMD, -1, d.pgamma, (float*)d.pD + t * TILE * TILE,
                  d.ptsum + t * TSUM_STRIDE, d.ptmax + t * TMAX_PER_TILE};
}

constexpr int HALF = TILE / 2;

// Epilogue through LDS, half a tile (64 rows) at a time, so a workgroup needs ~34 KB of LDS
// for it.  Row stride 132 floats: rows stay 16-byte aligned for vector reads, and the bank
// of (row, col) is (4 row + col) % 32, which the patterns below keep distinct within every
// 32 lanes.
constexpr int TILE_LDS = TILE + 4;

// Sums of a tile, in one order for every kernel:
//  row sums: four threads per row, thread q adding columns 32 q .. + 31 in order, then
//    (q 0 + q 1) + (q 2 + q 3);
//  column sums of a half tile (64 rows): for each h = 0, 1 the rows 8 i + 4 h .. + 3 (i < 4) of
//    the first and of the second 32 rows are added in order, then the two, then the two h --
//    the rows an MFMA accumulator's lane holds, so that they can be added in registers.
// Row sums of one row's quarter from LDS (a 16-byte boundary); cross tests keep the sums over
// the x2 columns (below `split`) and over the y2 columns apart.  Thread q writes for the row.
// Two batches of 16 entries, so that the accumulators may stay in registers beside them.
__device__ inline void emit_row(const BlockOut& o, int r, int q, const float* src, float& vmax) {
  double s0 = 0.0, s1 = 0.0;
#pragma unroll 1
  for (int b = 0; b < 32; b += 16) {
    float x[16];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float4 v = *(const float4*)(src + b + 4 * k);
      x[4 * k] = v.x; x[4 * k + 1] = v.y; x[4 * k + 2] = v.z; x[4 * k + 3] = v.w;
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) vmax = fmaxf(vmax, x[k]);  // block values are not negative
    if (o.split < 0) {
#pragma unroll
      for (int k = 0; k < 16; ++k) s0 += (double)x[k];
    } else {
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        const bool x2 = q * 32 + b + k < o.split;
        s0 += x2 ? (double)x[k] : 0.0;
        s1 += x2 ? 0.0 : (double)x[k];
      }
    }
  }
  s0 += __shfl_xor(s0, 1, 64);
  s0 += __shfl_xor(s0, 2, 64);
  if (q == 0) o.tsum[r] = s0;
  if (o.split < 0) return;
  s1 += __shfl_xor(s1, 1, 64);
  s1 += __shfl_xor(s1, 2, 64);
  if (q == 0) o.tsum[TILE + r] = s1;
}
// Column sum of one column of a half tile at `src` (two threads per column, h = 0 and 1, 32
// lanes apart).
__device__ inline void emit_col(const BlockOut& o, int half, int col, int h, const float* src) {
  double s = 0.0;
#pragma unroll 1
  for (int b = 0; b < 2; ++b) {
    float x[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) x[k] = src[(b * 32 + 8 * (k >> 2) + 4 * h + (k & 3)) * TILE_LDS];
    double t = 0.0;
#pragma unroll
    for (int k = 0; k < 16; ++k) t += (double)x[k];
    s = b ? s + t : t;
  }
  s += __shfl_xor(s, 32, 64);
  if (h == 0) o.tsum[TILE * (1 + half) + col] = s;
}

// Staged half tile (64 rows of block values) of a stored tile -> row sums, column sums, running
// max and stored rows.  All 256 threads take part.
__device__ inline void emit_half(const BlockOut& o, int half, const float* tl, float& vmax) {
  const int tid = threadIdx.x;
  emit_row(o, half * HALF + (tid >> 2), tid & 3, tl + (tid >> 2) * TILE_LDS + (tid & 3) * 32, vmax);
  const int col = (tid >> 6) * 32 + (tid & 31);
  emit_col(o, half, col, (tid >> 5) & 1, tl + col);
  float4* dst = (float4*)(o.D + half * HALF * TILE);
#pragma unroll
  for (int k = 0; k < HALF * TILE / 4 / 256; ++k) {
    const int f = tid + 256 * k;
    dst[f] = *(const float4*)(tl + (f >> 5) * TILE_LDS + 4 * (f & 31));
  }
}

// Near pairs: a Gram-based d^2 below 1e-3 of the norm sum has lost most of its digits to
// cancellation; such pairs (off the diagonal, inside the tile) are recomputed as a direct
// FP32 sum of squared differences of the input rows.
__device__ inline bool needs_refine(const TestDesc& d, const TileCtx& c, int r, int col,
                                    float d2, float nr, float nc) {
  return d.refine && r < c.rows_i && col < c.rows_j && !(c.diag && r == col) &&
         d2 < 1e-3f * (nr + nc);
}
__device__ inline float direct_d2(const TestDesc& d, const TileCtx& c, int r, int col) {
  const float* xa = input_row_f32(d, c.i, r);
  const float* xb = input_row_f32(d, c.j, col);
  float s = 0.0f;
  for (int k = 0; k < d.p; ++k) {
    const float df = xa[k] - xb[k];
    s = fmaf(df, df, s);
  }
  return s;
}
__device__ inline void add_refined(const TestDesc& d, int refined) {
  if (!refined) return;
  atomicAdd(&d.flags[1], refined);
  if (d.pflags) atomicAdd(&d.pflags[1], refined);
}

// Staged Gram entries of rows row0 .. row0 + rows - 1 of a tile -> block values of output o, in
// place, four adjacent columns at a time.  The loop is rolled and its near-pair path stands
// once: unrolled over a lane's accumulators it was 72 KB of code, whose instruction fetches took
// longer than the products of a small grid, and rolled over them (one entry at a time through
// indexed registers, a norm read and up to ten branches each) it took as long as the products of
// a large one.  edge: the tile has padding or the diagonal.
template <int THREADS>
__device__ inline void block_values(const TestDesc& d, const TileCtx& c, const BlockOut& o,
                                    int row0, int rows, bool edge, float* tl, const float* snorm,
                                    int& refined) {
#pragma unroll 1
  for (int f = threadIdx.x; f < rows * (TILE / 4); f += THREADS) {
    const int rl = f >> 5, c4 = 4 * (f & 31), r = row0 + rl;
    float4* q = (float4*)(tl + rl * TILE_LDS + c4);
    const float4 g = *q, n4 = *(const float4*)(snorm + TILE + c4);
    const float nv[4] = {n4.x, n4.y, n4.z, n4.w}, nr = snorm[r];
    float v[4] = {g.x, g.y, g.z, g.w};
    uint32_t near = 0u;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[e] = nr + nv[e] - 2.0f * v[e];
      if (v[e] < 1e-3f * (nr + nv[e])) near |= 1u << e;
    }
    while (near) {
      const int e = __builtin_ctz(near);
      near &= near - 1u;
      const float old = e == 0 ? v[0] : e == 1 ? v[1] : e == 2 ? v[2] : v[3];
      if (!needs_refine(d, c, r, c4 + e, old, nr, snorm[TILE + c4 + e])) continue;
      const float x = direct_d2(d, c, r, c4 + e);
      v[0] = e == 0 ? x : v[0];
      v[1] = e == 1 ? x : v[1];
      v[2] = e == 2 ? x : v[2];
      v[3] = e == 3 ? x : v[3];
      ++refined;
    }
    if (edge) {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = block_value_f32(o.kind, o.gamma, c, r, c4 + e, v[e]);
    } else if (o.kind == KIND_ED) {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = sqrtf(fmaxf(v[e], 0.0f));
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = expf((float)(-o.gamma) * fmaxf(v[e], 0.0f));
    }
    *q = make_float4(v[0], v[1], v[2], v[3]);
  }
}

// Correctly rounded square root of a float in [2^-96, 2^126]: the hardware's root s is within
// one ulp; the neighbour above is nearer when x lies past the midpoint, x - s^2 > s (up - s)
// (both sides multiples of the squared spacing, so the quarter term drops out), and likewise
// below.
__device__ inline float sqrt_rn(float x) {
  const float s = __builtin_amdgcn_sqrtf(x);
  const float up = __uint_as_float(__float_as_uint(s) + 1u);
  const float down = __uint_as_float(__float_as_uint(s) - 1u);
  const float r = fmaf(-s, s, x);
  const float v = r > s * (up - s) ? up : s;
  return r <= -(s * (s - down)) ? down : v;
}

typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));

// ------------------------------------------------------------------ tiles by an LDS ring
// F16: the staged operand holds fp16 pairs (hi, lo) of w 2^e (22 significant bits; see
// f16_split_exponent), and each Gram entry is formed as hi_a hi_b + hi_a lo_b + lo_a hi_b (the
// lo_a lo_b term, 2^-22 of the product, is dropped) with three v_mfma_f32_32x32x16_f16 into one
// FP32 accumulator: all three products are exact in FP32, so the entry carries the same FP32
// accumulation rounding as an FP32 Gram, at the fp16 MFMA rate.  The accumulator is scaled back
// by 2^-2e before the epilogue.  Else BF16 operands on v_mfma_f32_32x32x16_bf16.
//
// The operands go straight from the K-blocked staging into LDS (global_load_lds, one contiguous
// kilobyte per wave instruction): a stage is two 64-byte chunks of every row (fp16 pairs: 32
// coordinates; BF16: 64), NBUF stages make the ring, one barrier per stage.  Within a row the
// four 16-byte pieces of a chunk are stored at slot piece ^ ((row / 4) % 4), so that the 16
// lanes of a fragment read hit distinct bank groups.  Eight waves (2 x 4 of TR/2 x 32), two on
// every SIMD per workgroup: one wave's issue, waits and epilogue run under another's products.
// TR = 128: a stored tile per workgroup; TR = 64: half of one (64 rows x 128 columns).
//  - Grids of at most one workgroup per CU: a deep ring (NBUF 4 or 6), as there is no second
//    workgroup to hide the loads' latency, which leaves LDS for the split stream's workgroups
//    (16 KB each) beside it; half tiles while they fit.  (Whole tiles with NBUF 5: 35 instead of
//    36 us alone, but no room beside: FP32 MMD 344 + 2213 x 816 175 -> 162 us with 4.)
//  - Larger grids: NBUF 2; two whole tiles share a CU.
// Every shape adds an entry's products in the same order (chunk by chunk; hi hi, hi lo, lo hi)
// and forms values and sums alike, so all agree bit for bit, as does the super-tile kernel.
//
// The FP32 form's fp16 products run at 625 TFLOP/s at p = 1024 and 782 at p = 8192 on 528 tiles,
// whose last 16 make a second round of the 512 resident workgroups, and at 868 and 1000 on 2080
// tiles (85, 544, 241 and 1698 us; the library's 8192^3 product: 1111).  A launch of 528 tiles at p
// = 1000 keeps the matrix cores 25% busy.  Measured (FP32 form), against a kernel of four waves of
// 64 x 64 with register-staged 32-wide slices: 10 tiles at p = 1000 51 -> 20 us, 136 tiles at p =
// 512 38 -> 22 us, 256 tiles (cross test) at p = 1000 55 -> 36 us, 528 tiles at p = 1024 96 -> 84
// us, 7236 tiles at p = 512 (standard test) 461 -> 421 us (by this ring with four waves, three
// workgroups to a CU: 97 and 465).
//
// GATHER: rows staged once in their own order (standard test), read through the row map.
// first: the launch's first unit (a list past one dispatch goes in several).
constexpr int GR_THREADS = 512;
// WPE: waves per SIMD that the shape's workgroups per CU make.
// DUAL: a test of the launch may also write its MMD partner's blocks (the loop over both outputs
// keeps the accumulators live: 43 spilled registers, and 91 instead of 46 us on 1596 tiles at p =
// 32).
template <bool F16, int TR, int NBUF, int WPE, bool DUAL, bool GATHER = false>
__global__ void __launch_bounds__(GR_THREADS) __attribute__((amdgpu_waves_per_eu(WPE)))
k_gram_ring(const TestDesc* __restrict__ descs, const int64_t* __restrict__ offs, int ntests,
            int64_t first) {
  constexpr int THREADS = GR_THREADS, WAVES = THREADS / 64, WN = WAVES / 2;  // 2 x WN waves
  constexpr int MB = TR / 64;                    // 32-row blocks per wave (32 columns each)
  constexpr int NCH = 2;                         // chunks per stage
  constexpr bool REGS = TR == TILE;              // finish plain tiles in registers
  constexpr int NSTEP = NCH * (F16 ? 1 : 2);     // K steps of 16 per stage
  constexpr int NPL = F16 ? 2 : 1;               // operand halves per K step (F16: hi, lo)
  constexpr int NF = (TR + TILE) / 16;           // kilobyte loads per chunk
  constexpr int CHP = NF * 64;                   // 16-byte pieces per chunk
  constexpr int BUFP = NCH * CHP;                // pieces per stage
  constexpr int LOADS = NCH * NF / WAVES;        // loads per wave and stage
  constexpr int EPI = TR * TILE_LDS / 4;         // the epilogue's tile, in pieces
  constexpr int EPIP = EPI + 2 * TILE / 4 + 4;   // with the norms, flags and maxima
  static_assert(NCH * NF % WAVES == 0, "whole loads per wave");
  __shared__ __attribute__((aligned(16))) uint4 lds[NBUF * BUFP > EPIP ? NBUF * BUFP : EPIP];
  const int64_t u = first + xcd_grouped(blockIdx.x, gridDim.x);
  const int64_t bid = TR == TILE ? u : u >> 1;
  const int half = TR == TILE ? 0 : (int)(u & 1);
  const int ti_ = find_test(offs, ntests, bid);
  const TestDesc& d = descs[ti_];
  const TileCtx c = tile_ctx(d, bid - offs[ti_]);
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63,
            h = lane >> 5, lr = lane & 31;
  const int wm = w / WN, wn = w % WN;
  const int64_t nch = d.p_pad / (F16 ? 16 : 32);      // chunks per row, even
  const int64_t tstride = nch * TILE * CHUNK_HALVES;  // halves per staged tile
  const uint32_t piece = (uint32_t)(((lane & 3) ^ ((lane >> 4) & 3)) * 8);
  const uint32_t lane_src = (uint32_t)(lane >> 2) * CHUNK_HALVES + piece;
  const uint16_t* srcA = (const uint16_t*)d.W + c.i * tstride + half * HALF * CHUNK_HALVES + lane_src;
  const uint16_t* srcB = (const uint16_t*)d.W + c.j * tstride + lane_src;
  const int nst = (int)(nch / NCH);
  // load q of this wave and stage: chunk cc of rows 16 f .. + 15 (the TR rows, then the columns)
  const uint16_t* grow[GATHER ? LOADS : 1];
  if (GATHER) {
#pragma unroll
    for (int q = 0; q < LOADS; ++q) {
      const int f = (w * LOADS + q) % NF, rr = lane >> 2;
      const int64_t sr = f < TR / 16 ? staged_row(d, c.i, c.rows_i, half * HALF + f * 16 + rr)
                                     : staged_row(d, c.j, c.rows_j, (f - TR / 16) * 16 + rr);
      grow[GATHER ? q : 0] = (const uint16_t*)d.W + sr / TILE * tstride + (sr % TILE) * CHUNK_HALVES + piece;
    }
  }
  // the epilogue's norms and scale, loaded ahead of everything else
  float nreg = 0.0f;
  if (tid < 2 * TILE) {
    const int i = tid < TILE ? c.i : c.j, r = tid & (TILE - 1);
    nreg = ((const float*)d.nrm)[GATHER ? staged_row(d, i, tid < TILE ? c.rows_i : c.rows_j, r)
                                        : (int64_t)i * TILE + r];
  }
  const float unscale = F16 ? ldexpf(1.0f, -2 * f16_split_exponent(d)) : 1.0f;
  auto issue = [&](int st, int buf) {
#pragma unroll
    for (int q = 0; q < LOADS; ++q) {
      const int g = w * LOADS + q, cc = g / NF, f = g % NF;
      const uint16_t* src = GATHER ? grow[GATHER ? q : 0]
                            : f < TR / 16 ? srcA + f * (16 * CHUNK_HALVES)
                                          : srcB + (f - TR / 16) * (16 * CHUNK_HALVES);
      __builtin_amdgcn_global_load_lds(
          (const __attribute__((address_space(1))) void*)(src + (int64_t)(st * NCH + cc) *
                                                                    (TILE * CHUNK_HALVES)),
          (__attribute__((address_space(3))) void*)(lds + buf * BUFP + cc * CHP + f * 64), 16, 0, 0);
    }
  };
  typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
  const int sw = (lane >> 2) & 3;
  const int rd0 = lr * 4 + (h ^ sw);        // piece h       (BF16 first step; F16 hi)
  const int rd1 = lr * 4 + ((2 + h) ^ sw);  // piece 2 + h   (BF16 second step; F16 lo)
  u32x4 ca[MB * NPL], cb[NPL], na[MB * NPL], nb_[NPL];
  auto read = [&](int buf, int ks, u32x4 (&fa)[MB * NPL], u32x4 (&fb)[NPL]) {
    const uint4* base = lds + buf * BUFP + (F16 ? ks : ks >> 1) * CHP;
#pragma unroll
    for (int pl = 0; pl < NPL; ++pl) {
      const int rd = (F16 ? pl : ks & 1) ? rd1 : rd0;
#pragma unroll
      for (int m = 0; m < MB; ++m)
        fa[pl * MB + m] = __builtin_bit_cast(u32x4, base[(wm * MB + m) * 128 + rd]);
      fb[pl] = __builtin_bit_cast(u32x4, base[TR * 4 + wn * 128 + rd]);
    }
  };
  f32x16 acc[MB];
#pragma unroll
  for (int a = 0; a < MB; ++a)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[a][e] = 0.0f;
  // one K step's products; per accumulator the terms keep the order hi hi, hi lo, lo hi
  auto mfma = [&]() {
#pragma unroll
    for (int term = 0; term < (F16 ? 3 : 1); ++term)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        const u32x4 x = ca[(term == 2 ? MB : 0) + mb], y = cb[term == 1 ? 1 : 0];
        if (F16)
          acc[mb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(
              __builtin_bit_cast(f16x8_t, x), __builtin_bit_cast(f16x8_t, y), acc[mb], 0, 0, 0);
        else
          acc[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
              __builtin_bit_cast(bf16x8, x), __builtin_bit_cast(bf16x8, y), acc[mb], 0, 0, 0);
      }
  };
  // this wave's own reads have completed and its loads of stage st have landed (those of up to
  // NBUF - 2 later stages stay in flight); then everyone's
  auto arrive = [&](int st) {
    const int later = min(NBUF - 2, nst - 1 - st);
    __builtin_amdgcn_sched_barrier(0);
    // vmcnt in bits 3:0 and 15:14, expcnt not waited, lgkmcnt(0)
#define GR_WAIT(N) \
  __builtin_amdgcn_s_waitcnt(0x0070 | (((N) * LOADS) & 15) | ((((N) * LOADS) >> 4) << 14))
    static_assert((NBUF - 2) * LOADS < 64, "vmcnt");
    if (NBUF > 5 && later >= 4) GR_WAIT(NBUF > 5 ? 4 : 0);
    else if (NBUF > 4 && later >= 3) GR_WAIT(NBUF > 4 ? 3 : 0);
    else if (NBUF > 3 && later >= 2) GR_WAIT(NBUF > 3 ? 2 : 0);
    else if (later >= 1) GR_WAIT(1);
    else GR_WAIT(0);
#undef GR_WAIT
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll
  for (int q = 0; q < NBUF - 1; ++q)
    if (q < nst) issue(q, q);
  arrive(0);
  read(0, 0, ca, cb);
  int buf = 0;  // st % NBUF
  for (int st = 0; st < nst; ++st) {
    const int prev = buf == 0 ? NBUF - 1 : buf - 1, next = buf == NBUF - 1 ? 0 : buf + 1;
    if (st + NBUF - 1 < nst) issue(st + NBUF - 1, prev);  // stage st - 1's, read by all
#pragma unroll
    for (int ks = 0; ks < NSTEP; ++ks) {
      if (ks + 1 < NSTEP) {
        read(buf, ks + 1, na, nb_);
      } else if (st + 1 < nst) {
        arrive(st + 1);
        read(next, 0, na, nb_);
      }
      __builtin_amdgcn_sched_barrier(0);
      mfma();
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int k = 0; k < MB * NPL; ++k) ca[k] = na[k];
#pragma unroll
      for (int k = 0; k < NPL; ++k) cb[k] = nb_[k];
    }
    buf = next;
  }
  // ---- epilogue: block values, sums and maxima of the test's own output and (pD) of the MMD
  // test it feeds.  REGS: an energy-distance tile without near pairs or row norms outside
  // [2^-80, 2^99] (every d^2 then lies in sqrt_rn's range) is finished in registers: values,
  // column sums, maximum; its rows pass through LDS for the row sums and the coalesced store.
  // Otherwise (and on half tiles, where the 64 rows of a column's sum lie in two waves) the Gram
  // entries are staged and turned into values there.
  float* tl = (float*)lds;
  float* snorm = tl + EPI * 4;
  uint32_t* misc = (uint32_t*)(snorm + 2 * TILE);  // ok[4], near[8], maxima[2]
  const int col = wn * 32 + lr, row0 = wm * (TR / 2) + 4 * h;  // row0: in the workgroup's rows
  float* tcol = tl + row0 * TILE_LDS + col;  // entry (mb, e): row 32 mb + 8 (e / 4) + e % 4 on
  const bool edge = c.rows_i < TILE || c.rows_j < TILE || c.diag;
  __syncthreads();  // the ring is free
  if (tid < 2 * TILE) {
    snorm[tid] = nreg;
    const bool pad = (tid & (TILE - 1)) >= (tid < TILE ? c.rows_i : c.rows_j);
    const uint64_t ok = __ballot(pad || (nreg >= 0x1p-80f && nreg <= 0x1p99f));
    if (lane == 0) misc[w] = ok == ~0ull ? 1u : 0u;
  }
  if (tid < 2) misc[12 + tid] = 0u;
  bool fast = REGS && d.kind == KIND_ED;
  if (REGS && fast) {
    __syncthreads();  // norms staged
    // entry k = 32 mb + 8 g + u of this lane is row row0 + k (REGS: half == 0); padding and the
    // diagonal are never recomputed
    const int kend = col < c.rows_j ? c.rows_i - row0 : 0, kdiag = c.diag ? col - row0 : -1;
    const float nc = snorm[TILE + col];
    bool near = false;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float4 n4 = *(const float4*)(snorm + row0 + mb * 32 + 8 * g);
        const float nr[4] = {n4.x, n4.y, n4.z, n4.w};
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int k = mb * 32 + 8 * g + u;
          const float s = nr[u] + nc, gv = acc[mb][4 * g + u] * unscale;
          near |= k < kend && k != kdiag && s - 2.0f * gv < 1e-3f * s;
        }
      }
    const uint64_t anyn = __ballot(near);
    if (lane == 0) misc[4 + w] = anyn ? 1u : 0u;
    __syncthreads();
    fast = misc[0] & misc[1] & misc[2] & misc[3];
#pragma unroll
    for (int k = 0; k < WAVES; ++k) fast = fast && !misc[4 + k];
  }
  if (REGS && fast && !(DUAL && d.pD)) {
    const BlockOut o = own_out(d, c);
    const int kend = col < c.rows_j ? c.rows_i - row0 : 0, kdiag = c.diag ? col - row0 : -1;
    const float nc = snorm[TILE + col];
    float vmax = 0.0f;
    double cs[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      cs[mb] = 0.0;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float4 n4 = *(const float4*)(snorm + row0 + mb * 32 + 8 * g);
        const float nr[4] = {n4.x, n4.y, n4.z, n4.w};
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int k = mb * 32 + 8 * g + u;
          const float s = nr[u] + nc, gv = acc[mb][4 * g + u] * unscale;
          const float x = sqrt_rn(s - 2.0f * gv);
          const float v = k < kend && k != kdiag ? x : 0.0f;
          tcol[k * TILE_LDS] = v;
          vmax = fmaxf(vmax, v);
          cs[mb] += (double)v;
        }
      }
    }
    double s = cs[0] + cs[MB - 1];
    s += __shfl_xor(s, 32, 64);
    if (h == 0 && o.split < 0) o.tsum[TILE * (1 + wm) + col] = s;
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) vmax = fmaxf(vmax, __shfl_xor(vmax, m, 64));
    if (lane == 0) atomicMax(&misc[12], __float_as_uint(vmax));
    __syncthreads();
    if (tid == 0) {
      o.tmax[0] = __uint_as_float(misc[12]);
      o.tmax[1] = 0.0f;
    }
    float unused = 0.0f;
    emit_row(o, tid >> 2, tid & 3, tl + (tid >> 2) * TILE_LDS + (tid & 3) * 32, unused);
    if (o.D) {
      float4* dst = (float4*)o.D;
#pragma unroll
      for (int k = 0; k < TR * TILE / 4 / THREADS; ++k) {
        const int f = tid + THREADS * k;
        dst[f] = *(const float4*)(tl + (f >> 5) * TILE_LDS + 4 * (f & 31));
      }
    }
    return;
  }
#pragma nounroll
  for (int out = DUAL && d.pD ? 1 : 0; out >= 0; --out) {
    const BlockOut o = DUAL && out ? partner_out(d, c) : own_out(d, c);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int e = 0; e < 16; ++e)
        tcol[(mb * 32 + 8 * (e >> 2) + (e & 3)) * TILE_LDS] = acc[mb][e] * unscale;
    __syncthreads();
    int refined = 0;
    block_values<THREADS>(d, c, o, half * HALF, TR, edge, tl, snorm, refined);
    if (out == 0) add_refined(d, refined);
    __syncthreads();
    float vmax = 0.0f;
    if (tid < 4 * TR)
      emit_row(o, half * HALF + (tid >> 2), tid & 3, tl + (tid >> 2) * TILE_LDS + (tid & 3) * 32, vmax);
    if (o.split < 0) {
      // two threads per column and half (TR = 64: those without a row)
      const int t = TR == TILE ? tid : tid - 4 * TR;
      if (t >= 0) {
        const int hf = t >> 8, cl = ((t >> 6) & 3) * 32 + (t & 31);
        emit_col(o, half + hf, cl, (t >> 5) & 1, tl + hf * HALF * TILE_LDS + cl);
      }
      if (o.D) {
        float4* dst = (float4*)(o.D + half * HALF * TILE);
#pragma unroll
        for (int k = 0; k < TR * TILE / 4 / THREADS; ++k) {
          const int f = tid + THREADS * k;
          dst[f] = *(const float4*)(tl + (f >> 5) * TILE_LDS + 4 * (f & 31));
        }
      }
    }
    // non-negative floats order like their bit patterns
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) vmax = fmaxf(vmax, __shfl_xor(vmax, m, 64));
    if (lane == 0) atomicMax(&misc[12 + out], __float_as_uint(vmax));
    __syncthreads();  // (and the next output may stage)
    if (tid == 0) {
      o.tmax[half] = __uint_as_float(misc[12 + out]);
      if (TR == TILE) o.tmax[1] = 0.0f;
    }
  }
}

// ------------------------------------------------------- 256 x 256 workgroups (super tiles)
// One workgroup per 2 x 2 block of stored tiles: super tile (I, J) of the grid of
// ceil(nt / 2) super rows and columns (I <= J; for cross tests the rectangle of x-side by
// y-side super tiles).  Wave w = (a, b) = (w >> 1, w & 1) owns pooled tile
// (2I + a, 2J + b) and computes it whole with 4 x 4 accumulators of 32 x 32, so every A or
// B fragment it reads from LDS feeds four MFMAs (two in the 128-tile kernels), and the
// 256 operand rows of each side are fetched once per K slice for all four tiles.  The
// accumulators take a CU's whole register file, so one workgroup runs per CU; its epilogue
// could not overlap any MFMA work.  The kernel therefore ends with the raw Gram tile in the
// stored output tile, and k_gram_finish (one workgroup per stored tile, several per CU)
// forms the block values, sums and maxima.  A wave whose tile is not stored (the lower
// tile of a diagonal super tile, a tile past the edge of the grid) loads its share of the
// operands like the others; its products are discarded.
// (Cross tests, which store no block tile, are never planned on this kernel; the cross
// branch of super_tile keeps the layout consistent with the 128-tile kernels.)
struct SuperTile {
  // pooled tiles of the super row and column halves (-1: none) and the stored tile index
  // of each of the four tiles (-1: not stored); scalar fields with select accessors, so
  // that indexing by a runtime wave index does not move them to memory
  int ti0, ti1, tj0, tj1;
  int64_t t00, t01, t10, t11;
  __device__ int ti(int a) const { return a ? ti1 : ti0; }
  __device__ int tj(int b) const { return b ? tj1 : tj0; }
  __device__ int64_t tidx(int a, int b) const { return a ? (b ? t11 : t10) : (b ? t01 : t00); }
};

__device__ inline SuperTile super_tile(const TestDesc& d, int64_t local) {
  SuperTile s;
  int I, J;
  if (d.cross) {
    const int sy = (d.ty + 1) / 2;
    I = (int)(local / sy);
    J = (int)(local % sy);
    s.ti0 = 2 * I;
    s.ti1 = 2 * I + 1 < d.tx ? 2 * I + 1 : -1;
    s.tj0 = d.tx + 2 * J;
    s.tj1 = 2 * J + 1 < d.ty ? d.tx + 2 * J + 1 : -1;
    auto at = [&](int i, int j) -> int64_t {
      return i >= 0 && j >= 0 ? (int64_t)i * d.ty + (j - d.tx) : -1;
    };
    s.t00 = at(s.ti0, s.tj0);
    s.t01 = at(s.ti0, s.tj1);
    s.t10 = at(s.ti1, s.tj0);
    s.t11 = at(s.ti1, s.tj1);
  } else {
    tile_coords((int)local, (d.nt + 1) / 2, &I, &J);
    s.ti0 = 2 * I;
    s.ti1 = 2 * I + 1 < d.nt ? 2 * I + 1 : -1;
    s.tj0 = 2 * J;
    s.tj1 = 2 * J + 1 < d.nt ? 2 * J + 1 : -1;
    auto at = [&](int i, int j) -> int64_t {
      return i >= 0 && j >= 0 && i <= j ? tile_index(i, j, d.nt) : -1;
    };
    s.t00 = at(s.ti0, s.tj0);
    s.t01 = at(s.ti0, s.tj1);
    s.t10 = at(s.ti1, s.tj0);
    s.t11 = at(s.ti1, s.tj1);
  }
  return s;
}

__device__ inline TileCtx tile_ctx_at(const TestDesc& d, int i, int j, int64_t t) {
  TileCtx c;
  c.t = (int)t;
  c.i = i;
  c.j = j;
  c.rows_i = tile_rows(d, i);
  c.rows_j = tile_rows(d, j);
  c.diag = i == j;
  return c;
}

// Super-tile kernel.  F16 true: the staged operands are fp16 pairs (hi, lo) of the scaled
// centred values, three v_mfma_f32_32x32x16_f16 per product (hi hi, hi lo, lo hi); F16
// false: BF16 operands, v_mfma_f32_32x32x16_bf16.
//
// One K slice is one 64-byte chunk of every row (BF16: 32 coordinates, two K steps; fp16
// pairs: 16 coordinates, one K step, hi and lo).  In the K-blocked staging the chunks of
// 16 consecutive rows are one contiguous kilobyte, which one wave instruction moves
// straight into LDS (global_load_lds, 16 bytes per lane); each side of a slice is 256 rows
// x 64 bytes in LDS.  Within a row the four 16-byte pieces are stored at slot
// piece ^ ((row / 4) % 4), so that the 16 lanes of an MFMA fragment read (16 rows, one
// piece) hit 16 distinct bank groups; the loading lanes fetch their pieces in that permuted
// order, which keeps each load one contiguous kilobyte.  NBUF buffers of one slice each:
// the loads of slice s + NBUF are issued once slice s has been read, one barrier per slice.
template <bool F16>
__global__ void __launch_bounds__(256) k_gram_super(const TestDesc* __restrict__ descs,
                                                    const int64_t* __restrict__ offs,
                                                    int ntests) {
  constexpr int NSTEP = F16 ? 1 : 2;        // K steps of 16 per slice
  constexpr int NPL = F16 ? 2 : 1;          // operand halves per K step (F16: hi, lo)
  constexpr int SIDEP = 256 * 4;            // 16-byte pieces per side and slice
  constexpr int BUFP = 2 * SIDEP;           // pieces per buffer (both sides)
  constexpr int NBUF = 4;
  constexpr int LOADS = 2 * 16 / 4;         // kilobyte loads per wave and slice
  __shared__ __attribute__((aligned(16))) uint4 lds[NBUF * BUFP];
  const int64_t bid = xcd_grouped(blockIdx.x, gridDim.x);
  const int ti_ = find_test(offs, ntests, bid);
  const TestDesc& d = descs[ti_];
  const SuperTile st = super_tile(d, bid - offs[ti_]);
  // the wave index as a scalar, so that per-wave branches stay scalar branches
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63,
            h = lane >> 5, lr = lane & 31;
  const int wa = w >> 1, wb = w & 1;
  const bool active = __builtin_amdgcn_readfirstlane(st.tidx(wa, wb) >= 0 ? 1 : 0) != 0;
  f32x16 acc[4][4];
#pragma unroll
  for (int mb = 0; mb < 4; ++mb)
#pragma unroll
    for (int nb = 0; nb < 4; ++nb)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[mb][nb][e] = 0.0f;

  // Global sources.  Load f (of 32 per slice) is side f / 16, rows 16 (f % 16) .. + 15 of
  // that side's 256, which lie in its half (f % 16) / 8.  A half past the edge of the grid
  // reads the first half's rows: those products belong to waves whose tiles are not stored,
  // and are discarded.
  const int64_t nch = d.p_pad / (F16 ? 16 : 32);      // slices (chunks per row)
  const int64_t tstride = nch * TILE * CHUNK_HALVES;  // halves per staged tile
  const uint16_t* W = (const uint16_t*)d.W;
  // pooled tile of each side's halves (scalars; a missing half takes the first half's)
  const int tA0 = st.ti0, tA1 = st.ti1 >= 0 ? st.ti1 : st.ti0;
  const int tB0 = st.tj0, tB1 = st.tj1 >= 0 ? st.tj1 : st.tj0;
  // this lane's 16 bytes of a kilobyte load: row lane / 4 of the 16, stored at slot lane % 4,
  // which holds piece (lane % 4) ^ (row / 4) of that row
  const uint32_t lane_src = (uint32_t)(lane >> 2) * CHUNK_HALVES +
                            (uint32_t)(((lane & 3) ^ ((lane >> 4) & 3)) * 8);
  const uint16_t* srcA0 = W + tA0 * tstride + lane_src;
  const uint16_t* srcA1 = W + tA1 * tstride + lane_src;
  const uint16_t* srcB0 = W + tB0 * tstride + lane_src;
  const uint16_t* srcB1 = W + tB1 * tstride + lane_src;
  // issue the loads of slice SL into buffer BUF (this wave's LOADS kilobytes)
#define GS_ISSUE(SL, BUF)                                                                      \
  do {                                                                                         \
    _Pragma("unroll") for (int q = 0; q < LOADS; ++q) {                                        \
      const int f = w * LOADS + q, side = f >> 4, blk = f & 15;                                \
      const uint16_t* src = side ? ((blk >> 3) ? srcB1 : srcB0) : ((blk >> 3) ? srcA1 : srcA0); \
      __builtin_amdgcn_global_load_lds(                                                        \
          src + ((uint32_t)(SL) * (TILE * CHUNK_HALVES) + (uint32_t)(blk & 7) * (16 * CHUNK_HALVES)), \
          (__attribute__((address_space(3))) void*)(lds + (BUF) * BUFP + f * 64), 16, 0, 0);   \
    }                                                                                          \
  } while (0)
  typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
  const int nslices = (int)nch;
  // Fragment reads.  Row block rb (32 rows) of a side, K step ks, half pl: lane l reads row
  // rb * 32 + l % 32, piece (F16 ? 2 pl : 2 ks) + l / 32, at slot piece ^ ((l / 4) % 4).
  const int sw = (lane >> 2) & 3;
  const int rd0 = lr * 4 + ((h) ^ sw);           // piece h       (BF16 ks 0; F16 hi)
  const int rd1 = lr * 4 + ((2 + h) ^ sw);       // piece 2 + h   (BF16 ks 1; F16 lo)
#define GS_READ(BUF, KS, FA, FB)                                                              \
  do {                                                                                        \
    _Pragma("unroll") for (int pl = 0; pl < NPL; ++pl)                                        \
      _Pragma("unroll") for (int m = 0; m < 4; ++m) {                                         \
        const int rd_ = (F16 ? pl : (KS)) ? rd1 : rd0;                                        \
        FA[pl * 4 + m] = __builtin_bit_cast(                                                  \
            u32x4, lds[(BUF) * BUFP + (wa * 4 + m) * 128 + rd_]);                             \
        FB[pl * 4 + m] = __builtin_bit_cast(                                                  \
            u32x4, lds[(BUF) * BUFP + SIDEP + (wb * 4 + m) * 128 + rd_]);                     \
      }                                                                                       \
  } while (0)
  // wait until at most LATER slices of this wave's loads are in flight (vmcnt in bits 3:0
  // and 15:14; expcnt and lgkmcnt not waited)
#define GS_WAIT(LATER)                                                                        \
  do {                                                                                        \
    if ((LATER) >= 2)                                                                         \
      __builtin_amdgcn_s_waitcnt(0x0F70 | ((2 * LOADS) & 15) | (((2 * LOADS) >> 4) << 14));   \
    else if ((LATER) == 1)                                                                    \
      __builtin_amdgcn_s_waitcnt(0x0F70 | (LOADS & 15) | ((LOADS >> 4) << 14));               \
    else                                                                                      \
      __builtin_amdgcn_s_waitcnt(0x0F70);                                                     \
  } while (0)
  // A plain barrier: a fenced one would also wait for the loads of the later slices.
#define GS_BARRIER()                  \
  do {                                \
    __builtin_amdgcn_sched_barrier(0); \
    __builtin_amdgcn_s_barrier();      \
    __builtin_amdgcn_sched_barrier(0); \
  } while (0)
  // products of row blocks MB0 .. MB1 - 1 with the current fragments; per accumulator the
  // terms keep the order hi hi, hi lo, lo hi
#define GS_MFMA(MB0, MB1)                                                                   \
  do {                                                                                      \
    _Pragma("unroll") for (int mb = (MB0); mb < (MB1); ++mb)                                \
      _Pragma("unroll") for (int term = 0; term < (F16 ? 3 : 1); ++term)                    \
        _Pragma("unroll") for (int nb = 0; nb < 4; ++nb) {                                  \
          if (F16) {                                                                        \
            const f16x8_t x = __builtin_bit_cast(f16x8_t, ca[(term == 2 ? 4 : 0) + mb]);    \
            const f16x8_t y = __builtin_bit_cast(f16x8_t, cb[(term == 1 ? 4 : 0) + nb]);    \
            acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(x, y, acc[mb][nb], 0, 0, 0); \
          } else {                                                                          \
            acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(                          \
                __builtin_bit_cast(bf16x8, ca[mb]), __builtin_bit_cast(bf16x8, cb[nb]),     \
                acc[mb][nb], 0, 0, 0);                                                      \
          }                                                                                 \
        }                                                                                   \
  } while (0)
  // prologue: slices 0 .. NBUF - 1 in flight; wait for slice 0
#pragma unroll
  for (int u = 0; u < NBUF; ++u)
    if (u < nslices) GS_ISSUE(u, u);
  {
    const int later = min(NBUF - 1, nslices - 1);
    if (later >= 3)
      __builtin_amdgcn_s_waitcnt(0x0F70 | ((3 * LOADS) & 15) | (((3 * LOADS) >> 4) << 14));
    else
      GS_WAIT(later);
  }
  GS_BARRIER();
  u32x4 ca[4 * NPL], cb[4 * NPL], na[4 * NPL], nb_[4 * NPL];
  // Each K step: half the products; then the fragments of the next K step are read (at the
  // last step of a slice, after the slice boundary: own reads of slice sl complete, since
  // its buffer is refilled after the barrier; slice sl + 1 landed in every wave; slice
  // sl + NBUF issued); then the other half of the products, which run while those reads
  // are in flight.
  GS_READ(0, 0, ca, cb);
  for (int sl = 0; sl < nslices; ++sl) {
#pragma unroll
    for (int ks = 0; ks < NSTEP; ++ks) {
      GS_MFMA(0, 2);
      __builtin_amdgcn_sched_barrier(0);
      if (ks + 1 < NSTEP) {
        GS_READ(sl % NBUF, ks + 1, na, nb_);
      } else if (sl + 1 < nslices) {
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
        GS_WAIT(min(NBUF - 2, nslices - 2 - sl));
        GS_BARRIER();
        GS_READ((sl + 1) % NBUF, 0, na, nb_);
        __builtin_amdgcn_sched_barrier(0);
        if (sl + NBUF < nslices) GS_ISSUE(sl + NBUF, sl % NBUF);
      }
      __builtin_amdgcn_sched_barrier(0);
      GS_MFMA(2, 4);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int k = 0; k < 4 * NPL; ++k) {
        ca[k] = na[k];
        cb[k] = nb_[k];
      }
    }
  }
#undef GS_MFMA
#undef GS_READ
#undef GS_WAIT
#undef GS_BARRIER
#undef GS_ISSUE
  // ---- the raw Gram tile (times 2^(2 * scale_exp) for fp16 pairs), row-major, into the
  // stored output tile; k_gram_finish turns it into the test's block values
  if (active) {
    float* raw = (float*)d.D + st.tidx(wa, wb) * TILE * TILE;
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
      for (int nb = 0; nb < 4; ++nb)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int r = mb * 32 + 8 * (e >> 2) + 4 * h + (e & 3);
          raw[r * TILE + nb * 32 + lr] = acc[mb][nb][e];
        }
  }
}

// Finish of the super-tile Gram: one workgroup per stored tile turns the raw Gram tile
// into the test's block values (and, DUAL, those of the MMD test it feeds).  Each thread
// forms the squared distances of its 8 float4 of a half tile in registers as it loads them
// (the 128-tile kernels' expression d^2 = |a|^2 + |b|^2 - 2 g after the same exact
// power-of-two unscaling; near pairs, d^2 < 1e-3 (|a|^2 + |b|^2), recomputed as direct
// FP32 differences); each output's block values
// are then staged in LDS and emitted by the shared half-tile epilogue, so the outputs equal
// the 128-tile kernels' bit for bit.  Several workgroups share a CU (35 KB of LDS each),
// so this latency-bound pass overlaps itself.
template <bool DUAL>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(DUAL ? 3 : 4)))
k_gram_finish(const TestDesc* __restrict__ descs,
                                                     const int64_t* __restrict__ offs,
                                                     int ntests) {
  constexpr int NQ = HALF * TILE / 4 / 256;  // float4 per thread and half
  __shared__ __attribute__((aligned(16))) float tl[HALF * TILE_LDS];
  __shared__ float snorm[2 * TILE];
  __shared__ unsigned int tile_max_bits[2];
  const int64_t bid = xcd_grouped(blockIdx.x, gridDim.x);
  const int ti = find_test(offs, ntests, bid);
  const TestDesc& d = descs[ti];
  const TileCtx c = tile_ctx(d, bid - offs[ti]);
  const int tid = threadIdx.x;
  const float4* raw = (const float4*)((const float*)d.D + (int64_t)c.t * TILE * TILE);
  // entry f = tid + 256 k of a half: row f / 32, columns 4 (f % 32) .. + 3
  float4 cur[NQ];
#pragma unroll
  for (int k = 0; k < NQ; ++k) cur[k] = raw[tid + 256 * k];
  {
    const float* nrm = (const float*)d.nrm;
    snorm[tid] = nrm[(int64_t)(tid < TILE ? c.i : c.j) * TILE + (tid & (TILE - 1))];
  }
  if (tid < 2) tile_max_bits[tid] = 0u;
  const float unscale = d.gop == GOP_F16PAIR ? ldexpf(1.0f, -2 * f16_split_exponent(d)) : 1.0f;
  const bool has1 = DUAL && d.pD != nullptr;
  const BlockOut o0 = own_out(d, c), o1 = DUAL ? partner_out(d, c) : o0;
  float vmax0 = 0.0f, vmax1 = 0.0f;
  int refined = 0;
  __syncthreads();  // norms staged
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    if (half == 1) {
#pragma unroll
      for (int k = 0; k < NQ; ++k) cur[k] = raw[HALF * TILE / 4 + tid + 256 * k];
    }
    float dv[NQ][4];
    uint32_t near = 0u;  // bit 4 k + u: a near pair
#pragma unroll
    for (int k = 0; k < NQ; ++k) {
      const int f = tid + 256 * k, r = half * HALF + (f >> 5), c4 = 4 * (f & 31);
      const float g[4] = {cur[k].x, cur[k].y, cur[k].z, cur[k].w};
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const float nr = snorm[r], nc = snorm[TILE + c4 + u];
        dv[k][u] = nr + nc - 2.0f * (g[u] * unscale);
        if (needs_refine(d, c, r, c4 + u, dv[k][u], nr, nc)) near |= 1u << (4 * k + u);
      }
    }
#pragma nounroll
    for (int out = has1 ? 1 : 0; out >= 0; --out) {
      const BlockOut o = (DUAL && out) ? o1 : o0;
      const int kind = o.kind;
      const double gamma = o.gamma;
      __syncthreads();  // the previous emit has read tl
#pragma unroll
      for (int k = 0; k < NQ; ++k) {
        const int f = tid + 256 * k, r = half * HALF + (f >> 5), c4 = 4 * (f & 31);
        float v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = block_value_f32(kind, gamma, c, r, c4 + u, dv[k][u]);
        *(float4*)(tl + (f >> 5) * TILE_LDS + c4) = make_float4(v[0], v[1], v[2], v[3]);
      }
      // near pairs: values of the direct FP32 d^2 replace the staged ones
      uint32_t bits = near;
      while (bits) {
        const int b = __builtin_ctz(bits);
        bits &= bits - 1u;
        const int f = tid + 256 * (b >> 2), r = half * HALF + (f >> 5);
        const int col = 4 * (f & 31) + (b & 3);
        tl[(f >> 5) * TILE_LDS + col] =
            block_value_f32(kind, gamma, c, r, col, direct_d2(d, c, r, col));
        if (out == 0) ++refined;
      }
      __syncthreads();
      float vm = 0.0f;  // one emit call site: the maxima combine afterwards
      emit_half(o, half, tl, vm);
      if (DUAL && out) vmax1 = fmaxf(vmax1, vm);
      else vmax0 = fmaxf(vmax0, vm);
    }
  }
  add_refined(d, refined);
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) {
    vmax0 = fmaxf(vmax0, __shfl_xor(vmax0, m, 64));
    if (DUAL) vmax1 = fmaxf(vmax1, __shfl_xor(vmax1, m, 64));
  }
  // non-negative floats order like their bit patterns
  if ((tid & 63) == 0) {
    atomicMax(&tile_max_bits[0], __float_as_uint(vmax0));
    if (has1) atomicMax(&tile_max_bits[1], __float_as_uint(vmax1));
  }
  __syncthreads();
  if (tid == 0) {
    o0.tmax[0] = __uint_as_float(tile_max_bits[0]);
    o0.tmax[1] = 0.0f;
    if (has1) {
      o1.tmax[0] = __uint_as_float(tile_max_bits[1]);
      o1.tmax[1] = 0.0f;
    }
  }
}

// ---------------------------------------------------------------- FP64 direct
// Alg. 3 literally: sum over k of (x_ak - y_bk)^2 on the FP64 vector ALU, two instructions
// per pair and coordinate.  A workgroup computes 32 rows x 64 columns of a stored tile and
// its eight waves take an eighth of the coordinates each (4 of every 32), so that even the
// four tiles of a 200 + 200 test spread over 32 CUs with two waves on every SIMD; the eight
// partial sums are added in a fixed order at the end.  A lane holds 4 x 8 entries: per
// coordinate 12 8-byte LDS reads feed 64 FP64 instructions, which keeps the LDS below the
// vector ALU's time.  Rounds of 32 coordinates go straight into a ring of three LDS buffers
// (global_load_lds), two rounds ahead; the 16 pieces (two coordinates) of a staged row are
// stored at slot piece ^ (row % 8), so that the 8 rows of a fragment read lie in distinct
// banks.  Measured against one 128 x 128 tile per workgroup: 200 + 200 x 1000 (cross test,
// 4 tiles) 639 -> 46 us, latency-bound before and after; 1000 + 1000 x 500 303 -> 112 us (52
// us of vector-ALU time; four waves instead of eight took 107); 504 tiles of 90 + 33 rows, p =
// 25 (standard test) 45 -> 65 us, where a part's fixed cost (partial sums through LDS, root or
// exponential) is most of it, but the whole test 175 -> 165.
constexpr int DF_THREADS = 512;
constexpr int DF_ROWS = 32, DF_COLS = 64;      // entries of one workgroup
constexpr int DF_K = 32;                       // coordinates per round (4 per wave)
constexpr int DF_NBUF = 3;
constexpr int DF_BUF = (DF_ROWS + DF_COLS) * DF_K;  // doubles per buffer
constexpr int DF_PARTS = (TILE / DF_ROWS) * (TILE / DF_COLS);

// Block values, stored entries and sums of the rows lr + 8 (w % 4) and columns lc + 8 b +
// 32 (w / 4) of a 32 x 64 part: v[b] is the squared distance of that entry.  The sums of the
// row's 32 columns go to rs[0][w / 4] (cross tests: x2 columns there, y2 columns to rs[1]), the
// column sums of the wave's 8 rows to cs[w % 4].  Cross tests store no tile.
__device__ inline void dist_emit_f64(const TestDesc& d, const TileCtx& c, int r0, int c0, int w,
                                     int lane, const double (&v)[4], double (*rs)[2][32],
                                     double (*cs)[64]) {
  const int lr = lane >> 3, lc = lane & 7, hc = w >> 2;
  const int split = d.cross ? cross_split(d, c.j) : -1;
  const int r = r0 + 8 * (w & 3) + lr;
  double s0 = 0.0, s1 = 0.0, col[4];
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const int cc = c0 + lc + 8 * b + 32 * hc;
    double x;
    if (r >= c.rows_i || cc >= c.rows_j) x = 0.0;
    else if (c.diag && r == cc) x = d.kind == KIND_ED ? 0.0 : 1.0;
    else x = d.kind == KIND_ED ? sqrt(v[b]) : exp(-d.gamma * v[b]);
    if (split < 0 && d.D) ((double*)d.D)[(int64_t)c.t * TILE * TILE + r * TILE + cc] = x;
    if (split >= 0 && cc >= split) s1 += x;
    else s0 += x;
    col[b] = x;
  }
#pragma unroll
  for (int m = 1; m < 8; m <<= 1) {  // over the row's 8 lanes
    s0 += __shfl_xor(s0, m, 64);
    s1 += __shfl_xor(s1, m, 64);
  }
  if (lc == 0) {
    rs[0][hc][8 * (w & 3) + lr] = s0;
    if (split >= 0) rs[1][hc][8 * (w & 3) + lr] = s1;
  }
  if (split >= 0) return;
#pragma unroll
  for (int b = 0; b < 4; ++b) {  // over the wave's 8 rows
#pragma unroll
    for (int m = 8; m < 64; m <<= 1) col[b] += __shfl_xor(col[b], m, 64);
    if (lr == 0) cs[w & 3][lc + 8 * b + 32 * hc] = col[b];
  }
}

// GATHER: rows staged once in their own order (standard test), read through the row map.
template <bool GATHER>
__device__ inline void dist_part_f64(const TestDesc& d, const TileCtx& c, int part, double* sm) {
  constexpr int NLD = DF_BUF * 8 / 1024 / (DF_THREADS / 64);  // kilobyte loads per wave
  const int rq = part >> 1, ch = part & 1;
  const int r0 = rq * DF_ROWS, c0 = ch * DF_COLS;
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int lr = lane >> 3, lc = lane & 7;  // entries (lr + 8 a, lc + 8 b), a < 4, b < 8
  const double* Wa = (const double*)d.W + ((int64_t)c.i * TILE + r0) * d.p_pad;
  const double* Wb = (const double*)d.W + ((int64_t)c.j * TILE + c0) * d.p_pad;
  double* ts = d.tsum + (int64_t)c.t * d.tsum_stride;
  // a part that holds only padding: its entries are 0
  if (r0 >= c.rows_i || c0 >= c.rows_j) {
    if (tid < DF_ROWS) {
      ts[ch * TILE + r0 + tid] = 0.0;
      if (d.cross) ts[(2 + ch) * TILE + r0 + tid] = 0.0;
    }
    if (d.cross) return;
    if (tid < DF_COLS) ts[(2 + rq) * TILE + c0 + tid] = 0.0;
    if (d.D)
#pragma unroll
      for (int q = 0; q < DF_ROWS * DF_COLS / 2 / DF_THREADS; ++q) {
        const int e = 2 * (tid + DF_THREADS * q);
        *(double2*)((double*)d.D + (int64_t)c.t * TILE * TILE + (r0 + e / DF_COLS) * TILE + c0 +
                    e % DF_COLS) = make_double2(0.0, 0.0);
      }
    return;
  }
  const int nk = d.p_pad;
  // Load f = NLD w + q of a round moves staged rows 4 f .. + 3 (the 32 rows, then the 64
  // columns); this lane fills slot lane % 16 of row 4 f + lane / 16.
  const int row4 = lane >> 4;
  const int pk0 = 2 * ((lane & 15) ^ row4), pk1 = 2 * ((lane & 15) ^ (4 + row4));  // f even, odd
  const double* grow[GATHER ? NLD : 1];
  if (GATHER) {
#pragma unroll
    for (int q = 0; q < NLD; ++q) {
      const int row = 4 * (NLD * w + q) + row4;
      grow[GATHER ? q : 0] =
          (const double*)d.W + (row < DF_ROWS ? staged_row(d, c.i, c.rows_i, r0 + row)
                                              : staged_row(d, c.j, c.rows_j, c0 + row - DF_ROWS)) *
                                   d.p_pad;
    }
  }
  auto issue = [&](int round) {
#pragma unroll
    for (int q = 0; q < NLD; ++q) {
      const int f = NLD * w + q;
      const double* src = 4 * f < DF_ROWS ? Wa + (int64_t)4 * f * d.p_pad
                                          : Wb + (int64_t)(4 * f - DF_ROWS) * d.p_pad;
      // pieces past the row's end (never multiplied) read its last piece instead
      const int k = min(round * DF_K + ((f & 1) ? pk1 : pk0), nk - 2);
      __builtin_amdgcn_global_load_lds(
          (const __attribute__((address_space(1))) void*)(GATHER ? grow[q] + k
                                                                 : src + (uint32_t)(row4 * d.p_pad + k)),
          (__attribute__((address_space(3))) void*)(sm + (round % DF_NBUF) * DF_BUF + f * 128),
          16, 0, 0);
    }
  };
  double acc[4][8];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 8; ++b) acc[a][b] = 0.0;
  const int rounds = (nk + DF_K - 1) / DF_K;
#pragma unroll
  for (int r = 0; r < DF_NBUF - 1; ++r)
    if (r < rounds) issue(r);
  for (int r = 0; r < rounds; ++r) {
    // wait for this wave's loads of round r (those of round r + 1 stay in flight), then for
    // everyone's; the buffer of round r - 1, read by all, is refilled
    __builtin_amdgcn_sched_barrier(0);
    if (r + 1 < rounds) __builtin_amdgcn_s_waitcnt(0x0070 | NLD);  // vmcnt(NLD) lgkmcnt(0)
    else __builtin_amdgcn_s_waitcnt(0x0070);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    if (r + DF_NBUF - 1 < rounds) issue(r + DF_NBUF - 1);
    if (r * DF_K + 4 * w >= nk) continue;  // p_pad is a multiple of 16: whole groups of 4
    const double* A = sm + (r % DF_NBUF) * DF_BUF + lr * DF_K;
    const double* B = sm + (r % DF_NBUF) * DF_BUF + (DF_ROWS + lc) * DF_K;
#pragma unroll
    for (int k = 0; k < 4; ++k) {  // coordinate 4 w + k of the round, in piece 2 w + k / 2
      const int ao = 2 * ((2 * w + (k >> 1)) ^ lr) + (k & 1);
      const int bo = 2 * ((2 * w + (k >> 1)) ^ lc) + (k & 1);
      double av[4], bv[8];
#pragma unroll
      for (int a = 0; a < 4; ++a) av[a] = A[8 * a * DF_K + ao];
#pragma unroll
      for (int b = 0; b < 8; ++b) bv[b] = B[8 * b * DF_K + bo];
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 8; ++b) {
          const double df = av[a] - bv[b];
          acc[a][b] = fma(df, df, acc[a][b]);
        }
      if (k == 1) __builtin_amdgcn_sched_barrier(0);  // at most two coordinates' reads ahead
    }
  }
  // The waves' partial sums meet in LDS: waves 4..7 hand theirs to waves 0..3 (up to 16
  // coordinates they have none); then every wave finishes the rows lr + 8 (w % 4) of half of the
  // columns, from what waves 0..3 hand over.
  __syncthreads();
  if (nk > 16) {
    if (w >= 4) {
#pragma unroll
      for (int o = 0; o < 32; ++o) sm[((w - 4) * 32 + o) * 64 + lane] = acc[o >> 3][o & 7];
    }
    __syncthreads();
    if (w < 4) {
#pragma unroll
      for (int o = 0; o < 32; ++o) {
        acc[o >> 3][o & 7] += sm[(w * 32 + o) * 64 + lane];
        if (o % 8 == 7) __builtin_amdgcn_sched_barrier(0);  // at most eight reads ahead
      }
    }
    __syncthreads();
  }
  if (w < 4) {
#pragma unroll
    for (int o = 0; o < 32; ++o) sm[(w * 32 + o) * 64 + lane] = acc[o >> 3][o & 7];
  }
  __syncthreads();
  double v[4];
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const int o = 8 * (w & 3) + 4 * (w >> 2) + b;
    v[b] = 0.0;  // in the order of the waves
#pragma unroll
    for (int q = 0; q < 4; ++q) v[b] += sm[(q * 32 + o) * 64 + lane];
  }
  double (*rs)[2][32] = (double (*)[2][32])(sm + 4 * 32 * 64);
  double (*cs)[DF_COLS] = (double (*)[DF_COLS])(sm + 4 * 32 * 64 + 2 * 2 * 32);
  dist_emit_f64(d, c, r0, c0, w, lane, v, rs, cs);
  __syncthreads();
  if (tid < DF_ROWS) {
    ts[ch * TILE + r0 + tid] = rs[0][0][tid] + rs[0][1][tid];
    if (d.cross) ts[(2 + ch) * TILE + r0 + tid] = rs[1][0][tid] + rs[1][1][tid];
  }
  if (!d.cross && tid < DF_COLS)
    ts[(2 + rq) * TILE + c0 + tid] = (cs[0][tid] + cs[1][tid]) + (cs[2][tid] + cs[3][tid]);
}

// DF_PARTS units per stored tile.  first: the dispatch's first unit (one dispatch holds fewer than
// 2^32 work-items; a loop over units in the kernel had the constants of exp and sqrt hoisted out
// of it and 27 registers spilled).
template <bool GATHER>
__global__ void __launch_bounds__(DF_THREADS) __attribute__((amdgpu_waves_per_eu(4)))
k_dist_f64(const TestDesc* __restrict__ descs, const int64_t* __restrict__ offs, int ntests,
           int64_t first) {
  __shared__ __attribute__((aligned(16))) double sm[DF_NBUF * DF_BUF];
  static_assert(4 * 32 * 64 + 2 * 2 * 32 + 4 * DF_COLS <= DF_NBUF * DF_BUF,
                "the partial sums fit the operand buffers");
  const int64_t u = first + xcd_grouped(blockIdx.x, gridDim.x);
  const int64_t bid = u / DF_PARTS;
  const int ti = find_test(offs, ntests, bid);
  const TestDesc& d = descs[ti];
  dist_part_f64<GATHER>(d, tile_ctx(d, bid - offs[ti]), (int)(u % DF_PARTS), sm);
}
template <bool GATHER>
static void launch_dist_f64(int64_t blocks, hipStream_t st, const TestDesc* d, const int64_t* offs,
                            int n) {
  const int64_t units = blocks * DF_PARTS, most = 1 << 22;  // per dispatch
  for (int64_t first = 0; first < units; first += most)
    hipLaunchKernelGGL(k_dist_f64<GATHER>,
                       dim3((unsigned)(units - first < most ? units - first : most)),
                       dim3(DF_THREADS), 0, st, d, offs, n, first);
}

// Shape of a launch by its grid (stored tiles of all tests): half tiles while two workgroups per
// tile are at most one per CU; whole tiles with a deep ring up to one per CU (256 tiles at p =
// 1000: 36 us, half tiles three to a CU 44); whole tiles, two to a CU, beyond (990 tiles at p =
// 512 / 1024: 69 / 112 us, half tiles 77 / 128; 528 tiles 54 / 84, half tiles 49 / 79, but with
// the split stream beside them 91 against 104 at p = 1000).
constexpr int64_t GRAM_RING_MAX_HALVES = 128, GRAM_RING_MAX_TILES = 256;

template <bool F16, int TR, int NBUF, int WPE, bool DUAL, bool GATHER = false>
static void launch_ring_shape(int64_t blocks, hipStream_t st, const TestDesc* d,
                              const int64_t* offs, int n) {
  const int64_t units = TR == TILE ? blocks : 2 * blocks, most = 1 << 22;  // per dispatch
  for (int64_t first = 0; first < units; first += most)
    hipLaunchKernelGGL((k_gram_ring<F16, TR, NBUF, WPE, DUAL, GATHER>),
                       dim3((unsigned)(units - first < most ? units - first : most)),
                       dim3(GR_THREADS), 0, st, d, offs, n, first);
}
template <bool F16, bool DUAL>
static void launch_ring(int64_t blocks, hipStream_t st, const TestDesc* d, const int64_t* offs,
                        int n) {
  if (blocks <= GRAM_RING_MAX_HALVES)
    launch_ring_shape<F16, 64, 6, 2, DUAL>(blocks, st, d, offs, n);
  else if (blocks <= GRAM_RING_MAX_TILES)
    launch_ring_shape<F16, 128, 4, 2, DUAL>(blocks, st, d, offs, n);
  else
    launch_ring_shape<F16, 128, 2, 4, DUAL>(blocks, st, d, offs, n);
}
// dual: some test of the launch also writes its MMD partner's blocks (TestDesc::pD says which)
void launch_gram(int gop, bool super_tiles, int64_t blocks, hipStream_t st, const TestDesc* d,
                 const int64_t* offs, int n, bool dual) {
  if (blocks <= 0) return;
  const dim3 g((unsigned)blocks), b(256);
  if (super_tiles) {  // the raw Gram only; launch_gram_finish forms the block values
    if (gop == GOP_F16PAIR)
      hipLaunchKernelGGL(k_gram_super<true>, g, b, 0, st, d, offs, n);
    else if (gop == GOP_BF16)
      hipLaunchKernelGGL(k_gram_super<false>, g, b, 0, st, d, offs, n);
  } else if (gop == GOP_F64) {
    launch_dist_f64<false>(blocks, st, d, offs, n);
  } else if (gop == GOP_F16PAIR) {
    if (dual) launch_ring<true, true>(blocks, st, d, offs, n);
    else launch_ring<true, false>(blocks, st, d, offs, n);
  } else {
    if (dual) launch_ring<false, true>(blocks, st, d, offs, n);
    else launch_ring<false, false>(blocks, st, d, offs, n);
  }
}

// Tile sums of recomputations that share one staging (TestDesc::gather): `blocks` stored tiles.
void launch_gram_sums(int gop, int64_t blocks, hipStream_t st, const TestDesc* d,
                      const int64_t* offs, int n) {
  if (blocks <= 0) return;
  if (gop == GOP_F64)
    launch_dist_f64<true>(blocks, st, d, offs, n);
  else if (gop == GOP_F16PAIR)
    launch_ring_shape<true, 128, 2, 4, false, true>(blocks, st, d, offs, n);
  else
    launch_ring_shape<false, 128, 2, 4, false, true>(blocks, st, d, offs, n);
}

void launch_gram_finish(int64_t blocks, hipStream_t st, const TestDesc* d, const int64_t* offs,
                        int n, bool dual) {
  if (blocks <= 0) return;
  const dim3 g((unsigned)blocks), b(256);
  if (dual)
    hipLaunchKernelGGL(k_gram_finish<true>, g, b, 0, st, d, offs, n);
  else
    hipLaunchKernelGGL(k_gram_finish<false>, g, b, 0, st, d, offs, n);
}

}  // namespace et
