// The core of the int8 GEMM kernels (level_gemm_i8.hip, modular_gemm.hip): one 256 x 256
// output tile of sums of int8 products, by one workgroup of eight waves.
//
// Operands are k-contiguous rows of bytes (rows of A, columns of B), addressed by a base
// pointer, a row pitch and the walk of the stages copied.
//
// CDNA4 mapping:
// * v_mfma_i32_16x16x64_i8: lane l supplies 16 bytes of row l%16 of the A block
//   and of column l%16 of the B block, at k granule l/16 (any k order works as
//   long as A and B agree); register r of lane l holds D[4 (l/16) + r][l%16].
// * Eight waves (two per SIMD: one issues while the other waits; four waves of
//   128 x 128 ran 1-9% slower); each wave holds a 128 x 64 sub-tile in 32 accumulator
//   blocks (128 AGPRs).  The MFMAs are issued as inline instructions with AGPR
//   accumulators: left to itself the register allocator permutes accumulators between
//   AGPRs and VGPRs across the loop, dozens of copies per step that stall behind the
//   MFMAs writing them.
// * k advances in stages of 128 bytes, two LDS stages (64 KB each: the A tile
//   then the B tile, 128-byte rows).  Copies go global -> LDS directly with
//   buffer_load_dwordx4 ... lds (counted on vmcnt only; the FLAT form would make
//   the compiler wait for every LDS read).  A ds_read_b128 is served 16 lanes at
//   a time over 64 banks, lanes 8a .. 8a+7 together with 32+8a .. 32+8a+7 (the
//   grouping that the bank-conflict counter confirms: a swizzle conflict-free
//   for 16 consecutive lanes still doubled every read).  A fragment read meets
//   8 rows twice there, at granules g and g ^ 2, so the 16-byte granules of LDS
//   row R are XOR-swizzled by swz(R) = bit1(R) | (bit0(R) ^ bit3(R)) << 1 |
//   bit2(R) << 2, which keeps all 16 accesses on distinct bank groups (and 16
//   consecutive lanes too).
// * A stage is two sub-steps of 32 MFMAs per wave; the fragments of the next
//   sub-step are read (four groups of three ds_read_b128) while the current one
//   runs.  The barrier sits before a stage's last sub-step: it certifies the
//   next stage's copies and frees the current buffer, whose next copies (two
//   stages ahead) are then issued one pair after every eighth MFMA: a burst of
//   copies blocks the wave's in-order issue and starves the matrix pipe.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "internal.h"
#include "modular.h"

namespace mdg {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void lds_void;

constexpr int kTile = kModTile;
constexpr int kStage = kModStage;
constexpr int kBuf = 2 * kTile * kStage;  // one LDS stage: A tile then B tile
constexpr int kXcds = 8;
constexpr unsigned kWaitVmLgkm0 = 0x0070;  // s_waitcnt vmcnt(0) lgkmcnt(0)

// the granule swizzle of LDS row r (depends on r mod 16 only)
__device__ __forceinline__ int swz(int r) { return ((r >> 1) & 1) | ((((r & 1) ^ ((r >> 3) & 1))) << 1) | (r & 4); }

struct Frag {
  v4i a[8], b[4];
};

__device__ __forceinline__ void mfma(v4i& acc, const v4i& a, const v4i& b) {
  asm volatile("v_mfma_i32_16x16x64_i8 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}

// The position of the next copied stage: byte offsets into the rows of A and of B.
// kEven: the stages are an even number (the loop's single last stage takes 36 registers
// and spills beside the linear walk, 1% of the time).
struct Walk {
  static constexpr bool kEven = false;
  uint32_t a, b;        // current offsets
  uint32_t ja, jb;      // added at the end of a segment instead of kStage
  int within, spk;      // stage within the segment, stages per segment
  __device__ __forceinline__ void next() {
    const bool wrap = ++within == spk;
    a += wrap ? ja : kStage;
    b += wrap ? jb : kStage;
    within = wrap ? 0 : within;
  }
};

// The same for one run of stages in both operands.
struct Run {
  static constexpr bool kEven = true;
  uint32_t a;
  __device__ __forceinline__ void next() { a += kStage; }
};
__device__ __forceinline__ uint32_t offset_b(const Walk& w) { return w.b; }
__device__ __forceinline__ uint32_t offset_b(const Run& w) { return w.a; }

// The k loop of one tile.  The buffers are restrict parameters so that the
// LDS reads of one carry alias scopes that exclude the copies in flight into
// the other (the compiler then waits for neither).
template <class W>
__device__ __forceinline__ void tile_loop(int8_t* __restrict__ P0, int8_t* __restrict__ P1, const int8_t* a,
                                          const int8_t* b, uint32_t na, uint32_t nb, int nst, W walk, uint32_t qa,
                                          uint32_t qb, uint32_t la0, uint32_t la1, uint32_t lb0, uint32_t lb1,
                                          int fa0, int fa1, int fb0, int fb1, int wave, v4i (&acc)[8][4]) {
  const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t*>(a), 0, na, kBufferWord3);
  const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t*>(b), 0, nb, kBufferWord3);
  // copy q (0..3) of the walk's stage into buffer P: tile rows 32 wave + 8q .. +7 of A and of B
  auto copy = [&](int8_t* P, int q) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_void*)(P + (32 * wave + 8 * q) * kStage), 16, (q & 1) ? la1 : la0,
                                             walk.a + static_cast<uint32_t>(q) * qa, 0, 0);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (lds_void*)(P + kTile * kStage + (32 * wave + 8 * q) * kStage), 16,
                                             (q & 1) ? lb1 : lb0, offset_b(walk) + static_cast<uint32_t>(q) * qb, 0, 0);
  };
  auto read = [&](const int8_t* P, int h, Frag& f, int g) {
    const int oa = h ? fa1 : fa0, ob = h ? fb1 : fb0;
#pragma unroll
    for (int i = 2 * g; i < 2 * g + 2; ++i) f.a[i] = *reinterpret_cast<const v4i*>(P + oa + i * 16 * kStage);
    f.b[g] = *reinterpret_cast<const v4i*>(P + kTile * kStage + ob + g * 16 * kStage);
  };
  // rows 2g, 2g + 1 of the 8 x 4 blocks; with copies, copy pair g into P after the eighth MFMA
  auto run = [&](const Frag& f, int g, auto with_copies, int8_t* P) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int i = 2 * g + (e >> 2), j = e & 3;
      mfma(acc[i][j], f.a[i], f.b[j]);
      if constexpr (decltype(with_copies)::value) {
        if (e == 7) {
          __builtin_amdgcn_sched_barrier(0);
          copy(P, g);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
  };
  // sub-step: the next fragments (buffer Q, half h) into nxt while cur runs
  auto step = [&](const int8_t* Q, int h, Frag& nxt, const Frag& cur, auto with_copies, int8_t* P) {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      read(Q, h, nxt, g);
      __builtin_amdgcn_sched_barrier(0);
      run(cur, g, with_copies, P);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  Frag x, y;
  int left = nst;  // stages not yet copied
  // stage in buffer P (its sub-step 0 in x), the next one in Q; copies of the one
  // after that (near the end the last one again, into a buffer no one reads)
  auto stage = [&](int8_t* P, int8_t* Q) {
    step(P, 1, y, x, std::false_type{}, P);
    __builtin_amdgcn_s_waitcnt(kWaitVmLgkm0);  // this wave's copies of the next stage are in LDS, its reads of P done
    __syncthreads();                            // everyone's
    __builtin_amdgcn_sched_barrier(0);
    step(Q, 0, x, y, std::true_type{}, P);
    if (--left > 0) walk.next();
  };
  --left;
#pragma unroll
  for (int q = 0; q < 4; ++q) copy(P0, q);
  if (left > 0) walk.next();
  --left;
#pragma unroll
  for (int q = 0; q < 4; ++q) copy(P1, q);
  if (left > 0) walk.next();
  __builtin_amdgcn_s_waitcnt(kWaitVmLgkm0);
  __syncthreads();
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int g = 0; g < 4; ++g) read(P0, 0, x, g);
  int s = 0;
  for (; s + 1 < nst; s += 2) {
    stage(P0, P1);
    stage(P1, P0);
  }
  if constexpr (!W::kEven)
    if (s < nst) stage(P0, P1);
  // the last MFMAs' results settle before the accumulators are read, and the last
  // copies land before the block's LDS is given back
  asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" ::: "memory");
  __builtin_amdgcn_s_waitcnt(kWaitVmLgkm0);
}

// Where a block's tile and a lane's fragments and copies lie.
struct Tile {
  int64_t m0, n0;
  uint32_t la0, la1, lb0, lb1;  // copies: byte offsets of this lane from the tile's first row
  int fa0, fa1, fb0, fb1;       // fragments: LDS offsets
  int lane, wave, wr, wc;
};
__device__ __forceinline__ Tile tile_of(int64_t lda, int64_t ldb, int tiles_n, int ntiles, int group) {
  Tile t;
  // tile order: block b runs on XCD b % 8; XCD x takes the chunk [x per, (x+1) per)
  // of an order that walks patches of `group` tile-rows column by column
  int tt = blockIdx.x;
  {
    const int per = ntiles / kXcds;
    if (tt < per * kXcds) tt = (tt % kXcds) * per + tt / kXcds;
  }
  const int tiles_m = ntiles / tiles_n;
  const int gsz = group * tiles_n, g = tt / gsz, first = g * group;
  const int rows_in = min(group, tiles_m - first), within = tt - g * gsz;
  t.m0 = static_cast<int64_t>(first + within % rows_in) * kTile;
  t.n0 = static_cast<int64_t>(within / rows_in) * kTile;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  t.lane = lane;
  t.wave = wave;
  t.wr = wave >> 2;
  t.wc = wave & 3;
  // copies: lane L of instruction q lands at tile row 32 wave + 8q + L/8 (= 8 (q&1) + L/8
  // mod 16), granule L%8, and fetches logical granule (L%8) ^ swz(row) of that row
  const int lr = 32 * wave + (lane >> 3);
  const uint32_t g0 = static_cast<uint32_t>(((lane & 7) ^ swz(lane >> 3)) << 4);
  const uint32_t g1 = static_cast<uint32_t>(((lane & 7) ^ swz(8 + (lane >> 3))) << 4);
  const uint32_t ra = static_cast<uint32_t>(lr * lda), rb = static_cast<uint32_t>(lr * ldb);
  t.la0 = ra + g0;
  t.la1 = ra + g1;
  t.lb0 = rb + g0;
  t.lb1 = rb + g1;
  // fragments: lane l reads row 16 i + l%16 of the wave's 128 rows of A (64 columns of B),
  // logical granule 4h + l/16
  const int l = lane & 15;
  const int s0 = (((lane >> 4) ^ swz(l)) << 4) + l * kStage, s1 = (((4 + (lane >> 4)) ^ swz(l)) << 4) + l * kStage;
  t.fa0 = t.wr * 128 * kStage + s0;
  t.fa1 = t.wr * 128 * kStage + s1;
  t.fb0 = t.wc * 64 * kStage + s0;
  t.fb1 = t.wc * 64 * kStage + s1;
  return t;
}

__device__ __forceinline__ void clear(v4i (&acc)[8][4]) {
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = v4i{0, 0, 0, 0};
}

}  // namespace
}  // namespace mdg
