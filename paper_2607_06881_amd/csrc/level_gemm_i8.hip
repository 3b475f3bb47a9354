// Step a3 on the int8 matrix cores, hand-written: every level product of
// section 2 in one launch.
//
// The level G_t = sum over p + q = t of DA_p . DB_q is an integer sum of
// products of digits of at most 7 bits; the caller has checked that it stays
// below 2^31, so the int8 x int8 -> int32 matrix instruction forms it exactly
// in any order and blocking.
//
// Operands (written by the int8 splits): the digits of row i of A and of
// column j of B, k-contiguous, in rows of pitch ld = kI8Pad + S kp bytes:
//     DA  [mp][ld]: bytes kI8Pad + p kp + kk hold digit p of A[i][kk],
//     DBt [np][ld]: bytes kI8Pad + (S-1-q) kp + kk hold digit q of B[kk][j],
// zeros in the first kI8Pad bytes of every row and for kk >= k; kp is a
// multiple of 128, mp and np are m and n rounded up to 256 (rows beyond m or n
// only feed outputs that are not stored).  The pairs of level t are then one
// contiguous k range of length K = (p1 - p0 + 1) kp, starting at p0 kp in every
// row of DA and at (S-1-t+p0) kp in every row of DBt.  When K / 128 is odd the
// range starts one 128-byte stage early: that stage is the zero pad of A's row
// (p0 = 0) or of B's row (p0 > 0 means t >= S, so B's range starts at its pad),
// and adds nothing.  (Levels are split into chunks of pairs only when a pair is
// an even number of stages, so a chunk never needs that.)
//
// A tile is formed by the core of i8_core.h.
//
// Work decomposition: grid.x = output tiles (renumbered per XCD, as in the
// FP64 kernel, in patches of `group` tile-rows), grid.y = jobs, heaviest first
// (a table in the kernel arguments): whole levels, or, for small outputs whose
// grid would hold few blocks, chunks of a level's pairs that add their partial
// sums into zeroed planes with int32 atomics (exact in any order).
#include "i8_core.h"
#include "internal.h"

namespace mdg {
namespace {

static_assert(kI8Pad == kStage, "the zero pad is one stage");

// the jobs of one launch, heaviest first: level t[y], its pairs first[y] ..
// first[y] + count[y] - 1 (indices into the level's pair range)
struct Jobs {
  uint8_t t[128], first[128], count[128];
};

__global__ void __launch_bounds__(512, 1) level_gemm_i8_kernel(int64_t m, int64_t n, int64_t kp, int S, int tiles_n,
                                                               int ntiles, int group, const int8_t* __restrict__ DA,
                                                               const int8_t* __restrict__ DBt,
                                                               int32_t* __restrict__ G, Jobs jobs, int split) {
  __shared__ __attribute__((aligned(1024))) int8_t P0[kBuf];
  __shared__ __attribute__((aligned(1024))) int8_t P1[kBuf];

  const int t = jobs.t[blockIdx.y];
  const int p0 = (t - (S - 1) > 0 ? t - (S - 1) : 0) + jobs.first[blockIdx.y];
  const int64_t ld = kI8Pad + static_cast<int64_t>(S) * kp;
  int nst = static_cast<int>(jobs.count[blockIdx.y] * kp / kStage);
  const int odd = nst & 1;  // start one (zero) stage early
  nst += odd;
  const int64_t oa = kI8Pad + p0 * kp - odd * kStage, ob = kI8Pad + (S - 1 - t + p0) * kp - odd * kStage;
  const Tile tile = tile_of(ld, ld, tiles_n, ntiles, group);
  v4i acc[8][4];
  clear(acc);
  tile_loop(P0, P1, DA + tile.m0 * ld + oa, DBt + tile.n0 * ld + ob, static_cast<uint32_t>(kTile * ld - oa),
            static_cast<uint32_t>(kTile * ld - ob), nst, Run{0}, static_cast<uint32_t>(8 * ld),
            static_cast<uint32_t>(8 * ld), tile.la0, tile.la1, tile.lb0, tile.lb1, tile.fa0, tile.fa1, tile.fb0,
            tile.fb1, tile.wave, acc);

  int32_t* o = G + static_cast<int64_t>(t) * m * n;
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t gi = tile.m0 + tile.wr * 128 + i * 16 + 4 * (tile.lane >> 4) + r;
        const int64_t gj = tile.n0 + tile.wc * 64 + j * 16 + (tile.lane & 15);
        if (gi < m && gj < n) {
          if (split)
            atomicAdd(o + gi * n + gj, acc[i][j][r]);  // exact: the level's bound covers every partial sum
          else
            o[gi * n + gj] = acc[i][j][r];
        }
      }
}

__global__ void __launch_bounds__(256) zero_i32_kernel(int32_t* __restrict__ p, int64_t count) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < count; i += stride) p[i] = 0;
}

}  // namespace

bool level_gemm_i8_fits(int64_t kp, int S) {
  const int64_t ld = kI8Pad + static_cast<int64_t>(S) * kp;
  return S >= 1 && S <= kI8MaxSlices && kp > 0 && kp % kStage == 0 &&
         static_cast<int64_t>(kTile) * ld < (int64_t{1} << 31);
}

hipError_t launch_level_gemm_i8(int64_t m, int64_t n, int64_t kp, int S, int T, const int8_t* DA, const int8_t* DBt,
                                int32_t* G, hipStream_t stream) {
  if (m == 0 || n == 0) return hipSuccess;
  if (T < 0 || T > 2 * S - 2 || !level_gemm_i8_fits(kp, S)) return hipErrorInvalidValue;
  const int64_t tiles_m = (m + kTile - 1) / kTile, tiles_n = (n + kTile - 1) / kTile;
  const int64_t ntiles = tiles_m * tiles_n;
  if (ntiles > 0x7fffffff) return hipErrorInvalidValue;
  // Jobs: every level whole, or, when the grid would hold few blocks (small
  // outputs) and every pair is an even number of stages, each level split into
  // chunks of at most c pairs that add their sums into zeroed planes; heaviest
  // first (ties in level order).
  auto pairs_of = [&](int t) {
    const int p0 = t - (S - 1) > 0 ? t - (S - 1) : 0, p1 = t < S - 1 ? t : S - 1;
    return p1 - p0 + 1;
  };
  int chunk = S;
  const bool even = (kp / kStage) % 2 == 0;
  if (even && ntiles * (T + 1) < 512) {
    chunk = (S + 1) / 2;  // halves: on c1 (1024^2, S = 15) +11%; thirds and quarters lose to the atomics
    for (;; ++chunk) {
      int njobs = 0;
      for (int t = 0; t <= T; ++t) njobs += (pairs_of(t) + chunk - 1) / chunk;
      if (njobs <= 128) break;
    }
  }
  const bool split = chunk < S;
  Jobs jobs{};
  int cnt = 0;
  for (int size = chunk; size >= 1; --size)
    for (int t = 0; t <= T; ++t)
      for (int f = 0; f < pairs_of(t); f += chunk) {
        const int c = pairs_of(t) - f < chunk ? pairs_of(t) - f : chunk;
        if (c != size) continue;
        if (cnt == 128) return hipErrorInvalidValue;
        jobs.t[cnt] = static_cast<uint8_t>(t);
        jobs.first[cnt] = static_cast<uint8_t>(f);
        jobs.count[cnt] = static_cast<uint8_t>(c);
        ++cnt;
      }
  if (!split && cnt != T + 1) return hipErrorInvalidValue;
  if (split) {
    const int64_t count = static_cast<int64_t>(T + 1) * m * n;
    const int64_t blocks = (count + 255) / 256 < 4096 ? (count + 255) / 256 : 4096;
    hipLaunchKernelGGL(zero_i32_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, stream, G, count);
  }
  // patches of 2 tile-rows for large outputs, 4 otherwise (measured on MI355X)
  const int group = ntiles >= 1024 ? 2 : 4;
  hipLaunchKernelGGL(level_gemm_i8_kernel, dim3(static_cast<unsigned>(ntiles), static_cast<unsigned>(cnt)),
                     dim3(512), 0, stream, m, n, kp, S, static_cast<int>(tiles_n), static_cast<int>(ntiles), group,
                     DA, DBt, G, jobs, split ? 1 : 0);
  return hipGetLastError();
}

}  // namespace mdg
