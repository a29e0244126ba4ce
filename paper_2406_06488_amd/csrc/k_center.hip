// Double centring of the stored tiles.
//
// Adding f(a) + f(b) to every pooled pair leaves every resampled ED / MMD
// statistic unchanged: each pooled row of eq. (1)'s weights sums to zero
// (-nx/nx^2 + ny/(nx ny) = 0).  With f(a) = -r_a/n + R/(2 n^2), r_a the pooled
// row sum and R their total, the centred matrix has zero row sums, so for a
// split z (1 = member of x*)
//     ED*(z)  = -(1/nx + 1/ny)^2 * z^T Dc z,
//     MMD*(z) = +(1/nx + 1/ny)^2 * z^T Kc z,
// a single quadratic form over the three stored blocks.  Diagonal tiles are
// halved, so that z^T Dc z = 2 * sum over stored tiles (i <= j) of z_i^T T_ij z_j.
//
// FP32/BF16 forms: the centred value v, scaled by the test's power of two 2^e (so that
// |v| <= 2^14), becomes two planes whose products with split bits are exact:
//  FP32 form: hi = fp16(v), lo = fp16((v - hi) 2^11), multiplied by bits worth 1 and
//    2^-11: hi + lo 2^-11 holds v to about 2^-22 of itself;
//  BF16-refined form: hi = fp16(v), lo = e4m3((v - hi) 2^5) (|lo| <= 2^8 < 448), multiplied
//    by bits worth 1 and 2^-5 on the fp8 MFMA: v to about 2^-15 of itself, 3 bytes per entry.
// The hi (and fp16 lo) plane is laid out in v_mfma_f32_32x32x16_f16 A-fragment order:
// fragment (mb, ks) of a tile is 64 lanes x 8 values, lane = row%32 + 32 * ((col%16)/8),
// for rows 32 mb.. and columns 16 ks.. .  The e4m3 plane follows the 32x32x64 fp8
// A-fragment order: fragment (mb, kb) holds rows 32 mb.. and columns 64 kb.., lane
// row%32 + 32 * ((col%64)/32) holding 32 bytes (columns in order), stored as two 16-byte
// halves: [fragment][half][lane][16 bytes].
// FP64 form: one FP64 tile in the order v_mfma_f64_16x16x4f64 reads its A operand: fragment
// (rb, kp) holds rows 16 rb .. and columns 8 kp .., lane row%16 + 16 * ((col%8)/2) holding
// two adjacent columns (one for each of two instructions).
#include "e4m3.h"

namespace et {

// FP64 -> FP32, kept as a separate step: folded into the fp16 conversion that follows it,
// it would become one FP64 -> fp16 rounding, which has no hardware instruction.
__device__ inline float to_f32(double x) {
  float f = (float)x;
  asm volatile("" : "+v"(f));
  return f;
}

__device__ inline uint32_t pack_h2(_Float16 a, _Float16 b) {
  return (uint32_t)__builtin_bit_cast(uint16_t, a) | ((uint32_t)__builtin_bit_cast(uint16_t, b) << 16);
}

// One workgroup per half tile (rows 64 rh .. + 63: fragment row blocks 2 rh and 2 rh + 1),
// so that the grid has twice as many workgroups as stored tiles in flight; on grids
// planned with one workgroup per tile (past 2^22 tiles) a workgroup takes both halves.
__global__ void __launch_bounds__(256) k_center_split(const TestDesc* __restrict__ descs,
                                                      const int64_t* __restrict__ offs,
                                                      int ntests) {
  // centring constants of the tile's 128 rows and 128 columns (0 for padding)
  __shared__ double crow[TILE], ccol[TILE];
  const int ti = find_test(offs, ntests, blockIdx.x);
  const TestDesc d = descs[ti];
  const int64_t local = blockIdx.x - offs[ti];
  const bool halves = offs[ti + 1] - offs[ti] > d.ntiles;  // two workgroups per tile
  const int t = (int)(halves ? local >> 1 : local);
  const int rh0 = halves ? (int)(local & 1) : 0, rh1 = halves ? rh0 + 1 : 2;
  int i, j;
  tile_coords(t, d.nt, &i, &j);
  const int rows_i = tile_rows(d, i), rows_j = tile_rows(d, j);
  const double n = (double)d.nx + (double)d.ny;
  const double inv_n = 1.0 / n;
  const double c0 = d.obs[4] / (n * n);
  const double scale = d.obs[5];
  const double half = i == j ? 0.5 : 1.0;
  const bool f8lo = d.pfmt == PLANES_F16_E4M3;
  {
    const int r = threadIdx.x & (TILE - 1);
    const int blk = threadIdx.x < TILE ? i : j;
    const int64_t pa = (int64_t)blk * TILE + r;
    const double c = (d.rsum[pa * 2] + d.rsum[pa * 2 + 1]) * inv_n;
    if (threadIdx.x < TILE) crow[r] = c;
    else ccol[r] = c;
  }
  __syncthreads();
  const float* Dt = (const float*)d.D + (int64_t)t * TILE * TILE;
  uint8_t* P = (uint8_t*)d.planes + (int64_t)t * plane_bytes_per_entry(d.pfmt) * TILE * TILE;
  uint16_t* Phi = (uint16_t*)P;
  uint8_t* Plo = P + 2 * TILE * TILE;
  for (int rh = rh0; rh < rh1; ++rh) {
    // every load of the thread first (8 x 16 B in flight), then the conversions; fragment
    // q of the half: 8 values of row block q / 512 (2 rh or 2 rh + 1)
    constexpr int NQ = TILE * TILE / 8 / 256 / 2;
    float4 raw[NQ][2];
#pragma unroll
    for (int it = 0; it < NQ; ++it) {
      const int q = rh * (NQ * 256) + threadIdx.x + 256 * it;
      const int mb = q >> 9, ks = (q >> 6) & 7, lane = q & 63;
      const int r = mb * 32 + (lane & 31), c0l = ks * 16 + 8 * (lane >> 5);
      raw[it][0] = *(const float4*)(Dt + r * TILE + c0l);
      raw[it][1] = *(const float4*)(Dt + r * TILE + c0l + 4);
    }
#pragma unroll
    for (int it = 0; it < NQ; ++it) {
      const int q = rh * (NQ * 256) + threadIdx.x + 256 * it;
      const int mb = q >> 9, ks = (q >> 6) & 7, lane = q & 63;
      const int r = mb * 32 + (lane & 31), c0l = ks * 16 + 8 * (lane >> 5);
      const float v[8] = {raw[it][0].x, raw[it][0].y, raw[it][0].z, raw[it][0].w,
                          raw[it][1].x, raw[it][1].y, raw[it][1].z, raw[it][1].w};
      const double ca = crow[r];
      _Float16 hi[8], lo[8];
      float lo8[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int col = c0l + e;
        double x = 0.0;
        if (r < rows_i && col < rows_j) x = ((((double)v[e] - ca) - ccol[col]) + c0) * half * scale;
        // FP64 -> FP32 -> fp16 (both hardware conversions; a direct FP64 -> fp16 rounding is
        // a long software sequence): hi may then round one way twice, which the low plane
        // absorbs, since it is formed from the exact FP64 remainder x - hi
        hi[e] = (_Float16)to_f32(x);
        const double rem = x - (double)(float)hi[e];
        if (f8lo) lo8[e] = to_f32(rem * 32.0);
        else lo[e] = (_Float16)to_f32(rem * 2048.0);
      }
      uint4 w;
      w.x = pack_h2(hi[0], hi[1]); w.y = pack_h2(hi[2], hi[3]);
      w.z = pack_h2(hi[4], hi[5]); w.w = pack_h2(hi[6], hi[7]);
      *(uint4*)(Phi + (int64_t)q * 8) = w;
      if (f8lo) {
        // columns c0l .. c0l+7 are bytes (c0l % 16) .. +7 of half (c0l % 32) / 16 of lane
        // (r % 32) + 32 ((c0l % 64) / 32) in fragment (mb, c0l / 64)
        const int kb = c0l >> 6, g = (c0l >> 5) & 1, hf = (c0l >> 4) & 1;
        const int64_t off = ((int64_t)((mb * 2 + kb) * 2 + hf) * 64 + (lane & 31) + 32 * g) * 16 +
                            (c0l & 15);
        uint2 b;
        b.x = pack_e4m3(lo8);
        b.y = pack_e4m3(lo8 + 4);
        *(uint2*)(Plo + off) = b;
      } else {
        w.x = pack_h2(lo[0], lo[1]); w.y = pack_h2(lo[2], lo[3]);
        w.z = pack_h2(lo[4], lo[5]); w.w = pack_h2(lo[6], lo[7]);
        *(uint4*)(Phi + TILE * TILE + (int64_t)q * 8) = w;
      }
    }
  }
}

// One unit per 16-row fragment block of a stored tile, every load first (8 units per tile:
// with one workgroup per tile, 64 entries in turn per thread, three tiles took 14-20 us and
// 136 tiles 24 us, now 4 and 9); a grid smaller than the units strides over them.
constexpr int CF_PARTS = TILE / 16;
__global__ void __launch_bounds__(256) k_center_f64(const TestDesc* __restrict__ descs,
                                                    const int64_t* __restrict__ offs, int ntests,
                                                    int64_t units) {
  for (int64_t u = blockIdx.x; u < units; u += gridDim.x) {
    const int64_t bid = u / CF_PARTS;
    const int rb = (int)(u % CF_PARTS);
    const int ti = find_test(offs, ntests, bid);
    const TestDesc& d = descs[ti];
    const int t = (int)(bid - offs[ti]);
    int i, j;
    tile_coords(t, d.nt, &i, &j);
    const int rows_i = tile_rows(d, i), rows_j = tile_rows(d, j);
    const double n = (double)d.nx + (double)d.ny;
    const double inv_n = 1.0 / n;
    const double c0 = d.obs[4] / (n * n);
    const double half = i == j ? 0.5 : 1.0;
    // fragments kp = (threadIdx.x >> 6) + 4 s; this thread's row is the same in all of them
    const int lane = threadIdx.x & 63, r = rb * 16 + (lane & 15);
    const int64_t pa = (int64_t)i * TILE + r;
    const double ca = (d.rsum[pa * 2] + d.rsum[pa * 2 + 1]) * inv_n;
    const double* D = (const double*)d.D + (int64_t)t * TILE * TILE;
    double2* P = (double2*)((double*)d.planes + (int64_t)t * TILE * TILE) + rb * 16 * 64;
    double2 v[4], ra[4], rc[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int col = 8 * ((int)(threadIdx.x >> 6) + 4 * s) + 2 * (lane >> 4);
      v[s] = *(const double2*)(D + r * TILE + col);
      const double2* rs = (const double2*)(d.rsum + ((int64_t)j * TILE + col) * 2);
      ra[s] = rs[0];
      rc[s] = rs[1];
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int kp = (int)(threadIdx.x >> 6) + 4 * s, col = 8 * kp + 2 * (lane >> 4);
      const double cb0 = (ra[s].x + ra[s].y) * inv_n, cb1 = (rc[s].x + rc[s].y) * inv_n;
      double2 x = make_double2(0.0, 0.0);
      if (r < rows_i && col < rows_j) x.x = (((v[s].x - ca) - cb0) + c0) * half;
      if (r < rows_i && col + 1 < rows_j) x.y = (((v[s].y - ca) - cb1) + c0) * half;
      P[kp * 64 + lane] = x;
    }
  }
}

void launch_center(bool f64, int64_t blocks, hipStream_t st, const TestDesc* d,
                   const int64_t* offs, int n) {
  if (blocks <= 0) return;
  if (f64) {  // the launch table counts stored tiles
    const int64_t units = blocks * CF_PARTS;
    hipLaunchKernelGGL(k_center_f64, dim3((unsigned)(units < (1 << 23) ? units : (1 << 23))),
                       dim3(256), 0, st, d, offs, n, units);
  } else
    hipLaunchKernelGGL(k_center_split, dim3((unsigned)blocks), dim3(256), 0, st, d, offs, n);
}

}  // namespace et
