// Split stream: one lane per resampled split.
//
// Split b draws its nx members out of the n = nx + ny pooled items (X rows,
// then Y rows) by selection sampling (Knuth, TAOCP vol. 2, 3.4.2, Algorithm S):
// item t joins x* with probability need/(n - t), decided in integers as
// floor(u_t (n - t) / 2^64) < need, where u_t is a 64-bit Philox4x32-10 draw
// (Salmon et al., SC'11) with key (seed_lo, seed_hi) and counter
// (t/2, b_lo, b_hi, 0); even t uses output words (0, 1), odd t words (2, 3),
// low word first.  Once need is 0 (or equals the items left) the outcome is
// fixed and no draw is needed.  This replaces Alg. 2's SampleWithoutReplacement;
// the statistic only depends on which items form x*.
#include "common.h"

namespace et {

// Internal layout Z[w][col]: columns 0..B-1 drawn splits, B the identity split,
// the rest zero; words cover padded pooled positions (X tiles, then Y tiles).
//
// One workgroup serves MSPL consecutive split columns and walks the pooled
// tiles in order (one tile = 128 padded positions = 4 words).  The scaled draws
// v_t = floor(u_t (n - t) / 2^64) do not depend on the running count, so waves 1..3
// produce the next tile's draws into LDS while wave 0 runs the selection scan (one
// lane per split) over the current one.  Positions without an item (tile padding)
// hold v = 0xFFFFFFFF, which is never below need (< 2^31), so the scan is the same
// branch-free step for every position and writes whole words.
__device__ inline uint32_t scaled_draw(uint32_t lo, uint32_t hi, uint32_t m) {
  const uint64_t p_lo = (uint64_t)lo * m, p_hi = (uint64_t)hi * m;
  return (uint32_t)((p_hi + (p_lo >> 32)) >> 32);  // floor(u * m / 2^64), u = hi:lo
}

// The walk of one workgroup: MSPL splits from split number b0 (nb of them drawn), n items of
// which nx are members, in ntiles tiles of up to 128 items: tile_items(ch, &t_lo, &cnt) gives
// the items t_lo .. t_lo + cnt - 1 of tile ch, and put(ch, w, s, word) takes membership word w
// of tile ch of split b0 + s.
template <int MSPL, class Items, class Put>
__device__ __attribute__((always_inline)) inline void member_walk(
    uint32_t (*V)[TILE][MSPL], uint64_t seed, int64_t n, int64_t nx, uint64_t b0, int nb,
    int ntiles, Items tile_items, Put put) {
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
  auto draw_tile = [&](int ch, int buf, int first, int stride) {
    int64_t t_lo;
    int cnt;
    tile_items(ch, &t_lo, &cnt);
    // Philox counters t/2 covering the tile's items; a pair may straddle two tiles
    const int64_t c_lo = t_lo >> 1, c_hi = (t_lo + cnt - 1) >> 1;
    const int np = (int)(c_hi - c_lo + 1);
#pragma unroll 2
    for (int q = first; q < np * MSPL; q += stride) {
      const int s = q % MSPL;
      const int64_t ci = c_lo + q / MSPL;
      const uint64_t bb = b0 + (uint64_t)s;
      if (s >= nb) continue;
      const uint4 r = philox4x32_10(make_uint4((uint32_t)ci, (uint32_t)bb,
                                               (uint32_t)(bb >> 32), 0u), k0, k1);
      const int64_t t0 = 2 * ci;
      if (t0 >= t_lo) V[buf][t0 - t_lo][s] = scaled_draw(r.x, r.y, (uint32_t)(n - t0));
      if (t0 + 1 < t_lo + cnt)
        V[buf][t0 + 1 - t_lo][s] = scaled_draw(r.z, r.w, (uint32_t)(n - t0 - 1));
    }
    for (int q = first; q < (TILE - cnt) * MSPL; q += stride)
      V[buf][cnt + q / MSPL][q % MSPL] = 0xFFFFFFFFu;
  };
  draw_tile(0, 0, tid, MTHREADS);
  __syncthreads();
  // Selection scan.  Because v_t <= n - t - 1, the test v_t < need already keeps
  // every remaining item once need == n - t and none once need == 0.
  const bool drawn = lane < MSPL && lane < nb;
  uint32_t need = (uint32_t)nx;
  for (int ch = 0; ch < ntiles; ++ch) {
    if (wave != 0) {
      if (ch + 1 < ntiles) draw_tile(ch + 1, (ch + 1) & 1, tid - 64, MTHREADS - 64);
    } else if (drawn) {
      const uint32_t(*Vb)[MSPL] = V[ch & 1];
#pragma unroll
      for (int w = 0; w < TILE_WORDS; ++w) {
        uint32_t word = 0;
#pragma unroll
        for (int k8 = 0; k8 < 32; k8 += 8) {
          uint32_t v[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] = Vb[32 * w + k8 + e][lane];
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const uint32_t take = v[e] < need ? 1u : 0u;
            need -= take;
            word |= take << (k8 + e);
          }
        }
        put(ch, w, lane, word);
      }
    }
    __syncthreads();
  }
}

// MSPL is MEMBER_SPLITS, or MEMBER_SPLITS_WIDE for a launch with more workgroups than the
// chip holds at once: there the stream is bound by vector-ALU cycles, and a wider
// workgroup keeps twice as many of the scanning wave's lanes busy.
// At most 64 VGPRs, so that a wave of it fits on a SIMD beside four of the Gram's whole tiles
// (110 each), which it runs beside.
template <int MSPL>
__global__ void __launch_bounds__(MTHREADS) __attribute__((amdgpu_waves_per_eu(8)))
k_member(const TestDesc* __restrict__ descs, const int64_t* __restrict__ offs, int ntests) {
  __shared__ uint32_t V[2][TILE][MSPL];
  const int ti = find_test(offs, ntests, blockIdx.x);
  const TestDesc d = descs[ti];
  const int64_t col0 = (blockIdx.x - offs[ti]) * MSPL;
  const int tid = threadIdx.x;
  const int64_t n = (int64_t)d.nx + d.ny;
  const int xw = d.tx * TILE_WORDS, nwords = d.nt * TILE_WORDS;
  uint32_t* Z = d.Z;
  const int64_t BP = d.B_pad;
  // non-drawn columns: the identity split (column B) and zero padding
  if (col0 + MSPL > d.B) {
    for (int e = tid; e < nwords * MSPL; e += MTHREADS) {
      const int w = e / MSPL;
      const int64_t c = col0 + e % MSPL;
      if (c < d.B) continue;
      uint32_t v = 0;
      if (c == d.B && w < xw) {
        const int64_t cnt = d.nx - (int64_t)w * 32;
        v = cnt >= 32 ? 0xFFFFFFFFu : (cnt > 0 ? ((1u << cnt) - 1u) : 0u);
      }
      Z[(int64_t)w * BP + c] = v;
    }
  }
  if (col0 >= d.B) return;
  // pooled tile ch holds items t_lo .. t_lo + cnt - 1 at padded positions 0 .. cnt - 1
  auto tile_items = [&](int ch, int64_t* t_lo, int* cnt) {
    if (ch < d.tx) {
      *t_lo = (int64_t)ch * TILE;
      *cnt = (int)min<int64_t>(TILE, d.nx - *t_lo);
    } else {
      *t_lo = d.nx + (int64_t)(ch - d.tx) * TILE;
      *cnt = (int)min<int64_t>(TILE, n - *t_lo);
    }
  };
  member_walk<MSPL>(V, d.seed, n, d.nx, (uint64_t)col0, (int)min<int64_t>(MSPL, d.B - col0), d.nt,
                    tile_items, [&](int ch, int w, int s, uint32_t word) {
                      Z[(int64_t)(ch * TILE_WORDS + w) * BP + col0 + s] = word;
                    });
}

// Public layout: words[(b - b0) * W + t / 32], bit t % 32, W = ceil(n / 32); the same walk over
// the unpadded items (one thread per split took 192 us for 200 splits of 1000 items).
__global__ void __launch_bounds__(MTHREADS) k_member_public(int64_t nx, int64_t ny, uint64_t seed,
                                                            int64_t b0, int64_t count,
                                                            uint32_t* __restrict__ words) {
  __shared__ uint32_t V[2][TILE][MEMBER_SPLITS];
  const int64_t n = nx + ny, W = (n + 31) / 32;
  for (int64_t q0 = (int64_t)blockIdx.x * MEMBER_SPLITS; q0 < count;
       q0 += (int64_t)gridDim.x * MEMBER_SPLITS)
    member_walk<MEMBER_SPLITS>(
        V, seed, n, nx, (uint64_t)(b0 + q0), (int)min<int64_t>(MEMBER_SPLITS, count - q0),
        (int)((n + TILE - 1) / TILE),
        [&](int ch, int64_t* t_lo, int* cnt) {
          *t_lo = (int64_t)ch * TILE;
          *cnt = (int)min<int64_t>(TILE, n - *t_lo);
        },
        [&](int ch, int w, int s, uint32_t word) {
          const int64_t k = (int64_t)ch * TILE_WORDS + w;
          if (k < W) words[(q0 + s) * W + k] = word;
        });
}

// blocks: B_pad / MEMBER_SPLITS workgroups per test
void launch_member(int64_t blocks, hipStream_t st, const TestDesc* d, const int64_t* offs, int n,
                   bool wide) {
  if (blocks > 0)
    hipLaunchKernelGGL(wide ? k_member<MEMBER_SPLITS_WIDE> : k_member<MEMBER_SPLITS>,
                       dim3((unsigned)blocks), dim3(MTHREADS), 0, st, d, offs, n);
}
void launch_member_public(int64_t nx, int64_t ny, uint64_t seed, int64_t b0, int64_t count,
                          uint32_t* words, hipStream_t st) {
  if (count <= 0) return;
  const int64_t wg = (count + MEMBER_SPLITS - 1) / MEMBER_SPLITS;
  hipLaunchKernelGGL(k_member_public, dim3((unsigned)(wg < (1 << 20) ? wg : (1 << 20))),
                     dim3(MTHREADS), 0, st, nx, ny, seed, b0, count, words);
}

}  // namespace et
