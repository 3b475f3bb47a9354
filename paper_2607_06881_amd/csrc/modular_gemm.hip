// Step a3 for modular.h: all int8 products of a plan in one launch.
//
// Operands: int8 panels, k-contiguous, row i of A at DA + i lda holding panel p at
// p kp (B likewise by column), kp a multiple of 128, rows rounded up to 256
// (modular_split.hip).  A job sums nseg products of panels a + s da of A and
// b + s db of B, each kp long; every sum stays below 2^30 in magnitude, 2^29
// for residue jobs (checked by the planner), so the int8 x int8 -> int32 matrix
// instruction forms it exactly.
//
// A tile is formed by the core of i8_core.h.
//
// Epilogue: a lane's four accumulators of a block are four consecutive rows of
// one column.  Direct jobs store them as 16 bytes; residue jobs reduce each to y
// in [0, m] (floor division by a 32-bit multiply-high, exact below 2^29) and store
// four bytes, a quarter of the traffic.
#include <algorithm>

#include "i8_core.h"
#include "internal.h"
#include "modular.h"

namespace mdg {
namespace {

// the jobs of one launch: at most kJobsPerLaunch, longest first
constexpr int kJobsPerLaunch = 160;
struct Jobs {
  uint32_t j[kJobsPerLaunch][4];  // a | b << 16, da | db << 16, nseg | mod << 16, out (whole dwords for scalar loads)
};

__global__ void __launch_bounds__(512, 1) modular_gemm_kernel(int64_t m, int64_t n, int64_t kp, int64_t lda,
                                                              int64_t ldb, int tiles_n, int ntiles, int group,
                                                              const int8_t* __restrict__ DA,
                                                              const int8_t* __restrict__ DB,
                                                              uint32_t* __restrict__ P, Jobs jobs) {
  __shared__ __attribute__((aligned(1024))) int8_t P0[kBuf];
  __shared__ __attribute__((aligned(1024))) int8_t P1[kBuf];
  const Tile t = tile_of(lda, ldb, tiles_n, ntiles, group);
  ModJob job;
  {
    const uint32_t w0 = jobs.j[blockIdx.y][0], w1 = jobs.j[blockIdx.y][1], w2 = jobs.j[blockIdx.y][2];
    job.a = static_cast<uint16_t>(w0);
    job.b = static_cast<uint16_t>(w0 >> 16);
    job.da = static_cast<int16_t>(w1);
    job.db = static_cast<int16_t>(w1 >> 16);
    job.nseg = static_cast<uint16_t>(w2);
    job.mod = static_cast<uint16_t>(w2 >> 16);
    job.out = static_cast<uint16_t>(jobs.j[blockIdx.y][3]);
  }
  const int spk = static_cast<int>(kp / kStage), nst = spk * job.nseg;
  Walk walk;
  walk.a = static_cast<uint32_t>(job.a * kp);
  walk.b = static_cast<uint32_t>(job.b * kp);
  walk.ja = static_cast<uint32_t>(static_cast<int32_t>(job.da * kp - kp + kStage));
  walk.jb = static_cast<uint32_t>(static_cast<int32_t>(job.db * kp - kp + kStage));
  walk.within = 0;
  walk.spk = spk;

  v4i acc[8][4];
  clear(acc);
  tile_loop(P0, P1, DA + t.m0 * lda, DB + t.n0 * ldb, static_cast<uint32_t>(kTile * lda),
            static_cast<uint32_t>(kTile * ldb), nst, walk, static_cast<uint32_t>(8 * lda),
            static_cast<uint32_t>(8 * ldb), t.la0, t.la1, t.lb0, t.lb1, t.fa0, t.fa1, t.fb0, t.fb1, t.wave, acc);

  const int64_t quads = (m + 3) / 4, unit = quads * n;
  const int64_t q0 = t.m0 / 4 + t.wr * 32 + (t.lane >> 4), j0 = t.n0 + t.wc * 64 + (t.lane & 15);
  if (job.mod == kDirectJob) {
    v4i* o = reinterpret_cast<v4i*>(P + job.out * unit);
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int64_t gq = q0 + 4 * i, gj = j0 + 16 * j;
        if (gq < quads && gj < n) o[gq * n + gj] = acc[i][j];
      }
  } else {
    const int md = kModuli[job.mod];
    // ceil(2^37 / m), below 2^31 for m > 64: x magic / 2^37 exceeds x / m by less than
    // 1 / m in magnitude for |x| < 2^29, so its floor is floor(x / m), except one less
    // at negative multiples of m (then y = m, the same residue; m = 256 is exact)
    const int magic = static_cast<int>(((uint64_t{1} << 37) + md - 1) / md);
    uint32_t* o = P + job.out * unit;
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        uint32_t w = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int x = acc[i][j][r];
          const int q = __mulhi(x, magic) >> 5;  // below 2^23 in magnitude
          const uint32_t y = static_cast<uint32_t>(x + __mul24(q, -md)) & 0xffu;
          w |= y << (8 * r);
        }
        const int64_t gq = q0 + 4 * i, gj = j0 + 16 * j;
        if (gq < quads && gj < n) o[gq * n + gj] = w;
      }
  }
}

// An offset beyond every plane's buffer (at most 2^31 bytes, kLevelsMaxN), also with a
// column step added.  The steps go into the offset that the hardware checks, not into the
// scalar one: the check is against the size minus the scalar offset, which is below zero
// for a last tile of fewer than 48 elements (say 1 row, 1 column).
constexpr uint32_t kOutside = 0xfffff000u;
typedef uint32_t v2u __attribute__((ext_vector_type(2)));

// The levels of a LevelPlan: blockIdx.y is the position in `order` (heaviest level
// first, a byte each).  Every pass reads the sums of the ones before it back from
// the level's own plane (int64 until the last), which the same thread wrote.
struct Levels {
  int S, c;
  uint32_t order[(kMaxLevels + 3) / 4];
};
__global__ void __launch_bounds__(512, 1) modular_levels_kernel(int64_t m, int64_t n, int64_t kp, int64_t ld,
                                                                int tiles_n, int ntiles, int group,
                                                                const int8_t* __restrict__ DA,
                                                                const int8_t* __restrict__ DB, double* __restrict__ G,
                                                                Levels levels) {
  __shared__ __attribute__((aligned(1024))) int8_t P0[kBuf];
  __shared__ __attribute__((aligned(1024))) int8_t P1[kBuf];
  const Tile t = tile_of(ld, ld, tiles_n, ntiles, group);
  const int level = (levels.order[blockIdx.y >> 2] >> (8 * (blockIdx.y & 3))) & 0xffu;
  const int S = levels.S, c = levels.c;
  const int p0 = level - (S - 1) > 0 ? level - (S - 1) : 0, p1 = level < S - 1 ? level : S - 1;
  const int spk = static_cast<int>((p1 - p0 + 1) * kp / kStage);  // a run: the level's pairs for one (i, j)
  // the tile's rows of the plane as a buffer, whose range check drops the rows beyond
  // m; the columns beyond n get an offset outside of it
  const uint32_t pitch = static_cast<uint32_t>(n * 8);
  const __amdgpu_buffer_rsrc_t rg = __builtin_amdgcn_make_buffer_rsrc(
      G + (static_cast<int64_t>(level) * m + t.m0) * n, 0,
      static_cast<uint32_t>(m - t.m0 < kTile ? m - t.m0 : kTile) * pitch, kBufferWord3);
  const int64_t j0 = t.n0 + t.wc * 64 + (t.lane & 15);
  const uint32_t off0 = static_cast<uint32_t>(t.wr * 128 + 4 * (t.lane >> 4)) * pitch + static_cast<uint32_t>(j0 * 8);
  const int cols = j0 >= n ? 0 : static_cast<int>((n - j0 + 15) / 16 < 4 ? (n - j0 + 15) / 16 : 4);  // of the lane's 4
  for (int s = 0; s <= 2 * c - 2; ++s) {
    const int i = s - (c - 1) > 0 ? s - (c - 1) : 0, runs = min(s, c - 1) - i + 1;
    Walk walk;
    walk.a = static_cast<uint32_t>((i * S + p0) * kp);
    walk.b = static_cast<uint32_t>(((s - i) * S + S - 1 - level + p0) * kp);
    walk.ja = static_cast<uint32_t>(static_cast<int32_t>(S * kp) - (spk - 1) * kStage);
    walk.jb = static_cast<uint32_t>(-static_cast<int32_t>(S * kp) - (spk - 1) * kStage);
    walk.within = 0;
    walk.spk = spk;
    v4i acc[8][4];
    clear(acc);
    tile_loop(P0, P1, DA + t.m0 * ld, DB + t.n0 * ld, static_cast<uint32_t>(kTile * ld),
              static_cast<uint32_t>(kTile * ld), runs * spk, walk, static_cast<uint32_t>(8 * ld),
              static_cast<uint32_t>(8 * ld), t.la0, t.la1, t.lb0, t.lb1, t.fa0, t.fa1, t.fb0, t.fb1, t.wave, acc);
    const bool last = s == 2 * c - 2;
    // 16 elements at a time: their loads are in flight together, and the offsets,
    // formed anew in every pass, leave the accumulators their registers
    uint32_t off = off0;
    asm volatile("" : "+v"(off));
#pragma unroll
    for (int x = 0; x < 8; ++x) {
      v2u old[4][4];
      if (s > 0) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int y = 0; y < 4; ++y)
            old[r][y] =
                __builtin_amdgcn_raw_buffer_load_b64(rg, (y < cols ? off + r * pitch : kOutside) + 128 * y, 0, 0);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int y = 0; y < 4; ++y) {
          int64_t v = static_cast<int64_t>(acc[x][y][r]) << (7 * s);
          if (s > 0) v += static_cast<int64_t>(old[r][y][0] | static_cast<uint64_t>(old[r][y][1]) << 32);
          if (last) v = __double_as_longlong(static_cast<double>(v));  // below 2^53: exact
          const v2u d = {static_cast<uint32_t>(v), static_cast<uint32_t>(v >> 32)};
          __builtin_amdgcn_raw_buffer_store_b64(d, rg, (y < cols ? off + r * pitch : kOutside) + 128 * y, 0, 0);
        }
      off += 16 * pitch;
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

}  // namespace

hipError_t launch_modular_levels(int64_t m, int64_t n, int64_t kp, const LevelPlan& lp, const int8_t* DA,
                                 const int8_t* DB, double* G, hipStream_t stream) {
  if (m == 0 || n == 0) return hipSuccess;
  const int panels = lp.c * lp.S;
  if (!modular_gemm_fits(kp, panels) || lp.T + 1 > kMaxLevels || n > kLevelsMaxN) return hipErrorInvalidValue;
  const int64_t tiles_m = (m + kTile - 1) / kTile, tiles_n = (n + kTile - 1) / kTile;
  const int64_t ntiles = tiles_m * tiles_n;
  if (ntiles > 0x7fffffff) return hipErrorInvalidValue;
  Levels lv{};
  lv.S = lp.S;
  lv.c = lp.c;
  int at = 0;
  for (int size = lp.S; size >= 1; --size)
    for (int t = 0; t <= lp.T; ++t) {
      const int lo = std::max(0, t - (lp.S - 1)), hi = std::min(t, lp.S - 1);
      if (hi - lo + 1 != size) continue;
      lv.order[at >> 2] |= static_cast<uint32_t>(t) << (8 * (at & 3));
      ++at;
    }
  const int group = ntiles >= 1024 ? 2 : 4;
  hipLaunchKernelGGL(modular_levels_kernel, dim3(static_cast<unsigned>(ntiles), static_cast<unsigned>(lp.T + 1)),
                     dim3(512), 0, stream, m, n, kp, panels * kp, static_cast<int>(tiles_n),
                     static_cast<int>(ntiles), group, DA, DB, G, lv);
  return hipGetLastError();
}

bool modular_gemm_fits(int64_t kp, int panels) {
  return panels >= 1 && kp > 0 && kp % kStage == 0 && static_cast<int64_t>(kTile) * panels * kp < (int64_t{1} << 31);
}

hipError_t launch_modular_gemm(int64_t m, int64_t n, int64_t kp, const ModPlan& pl, const int8_t* DA, const int8_t* DB,
                               uint32_t* P, hipStream_t stream) {
  if (m == 0 || n == 0) return hipSuccess;
  if (!modular_gemm_fits(kp, pl.pa) || !modular_gemm_fits(kp, pl.pb)) return hipErrorInvalidValue;
  const int64_t tiles_m = (m + kTile - 1) / kTile, tiles_n = (n + kTile - 1) / kTile;
  const int64_t ntiles = tiles_m * tiles_n;
  if (ntiles > 0x7fffffff) return hipErrorInvalidValue;
  // patches of 2 tile-rows for large outputs, 4 otherwise (measured on MI355X)
  const int group = ntiles >= 1024 ? 2 : 4;
  for (size_t first = 0; first < pl.jobs.size(); first += kJobsPerLaunch) {
    const size_t count = std::min<size_t>(kJobsPerLaunch, pl.jobs.size() - first);
    Jobs jobs{};
    for (size_t i = 0; i < count; ++i) {
      const ModJob& j = pl.jobs[first + i];
      jobs.j[i][0] = j.a | static_cast<uint32_t>(j.b) << 16;
      jobs.j[i][1] = static_cast<uint16_t>(j.da) | static_cast<uint32_t>(static_cast<uint16_t>(j.db)) << 16;
      jobs.j[i][2] = j.nseg | static_cast<uint32_t>(j.mod) << 16;
      jobs.j[i][3] = j.out;
    }
    hipLaunchKernelGGL(modular_gemm_kernel, dim3(static_cast<unsigned>(ntiles), static_cast<unsigned>(count)),
                       dim3(512), 0, stream, m, n, kp, pl.pa * kp, pl.pb * kp, static_cast<int>(tiles_n),
                       static_cast<int>(ntiles), group, DA, DB, P, jobs);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace mdg
