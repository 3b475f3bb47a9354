// Step a2 for the int8 products of modular.h: the digits of every element, as
// one integer D per element (digits.h), turned into int8 panels: balanced
// residues of blocks of digits, and the 7-bit sub-digits (and their pairwise
// sums) of single digits.
//
// Panels are k-contiguous: row `line` (a row of A or a column of B) holds its
// panels one after the other, kp = k rounded up to 128 bytes each, zeros for
// kk >= k.  A block of threads takes 16 lines x TK values of k: the limbs go
// through LDS, so that global loads are whole 128-byte lines for both operands
// (A's lines are rows, B's are columns), and every thread then turns four
// consecutive k of one line into panel bytes, stored as one dword: a wave stores
// 64 or 128 contiguous bytes of each line per panel.
//
// A residue is formed from the block's bytes: x = sum of byte_j (256^j f mod m),
// with v_dot4_u32_u8 on four bytes at a time (f = 1, or W_i^-1 mod m_i for A), x
// below 2^21, then x - m rint(x / m) in float (exact: integers below 2^24), which
// lies in [-m/2, m/2]; the sign of the element multiplies it.  Bound by HBM
// (8 L bytes read and one byte per panel written per element) together with about
// nine vector operations per panel and element.
//
// Both operands go in one launch, and where that has fewer than 512 blocks, the
// panels are shared out over up to eight blocks per tile (grid.z), each splitting
// the tile again: a tile's panels are one serial chain of scalar loads and vector
// work per wave (20 us per operand at 333 x 501 with one block per tile).
#include <algorithm>

#include "digits.h"
#include "internal.h"
#include "modular.h"
#include "modular_tables.h"

namespace mdg {
namespace {

constexpr int kLines = kModSplitLines;

__constant__ const ResidueTable kResidueTable = make_residue_table();

// The blocks in one dword each (scalar loads need whole, aligned dwords).
inline uint32_t pack_block(const ModBlock& b) {
  return b.lo | static_cast<uint32_t>(b.bits) << 10 | static_cast<uint32_t>(b.count) << 18 |
         static_cast<uint32_t>(b.residue) << 24 | static_cast<uint32_t>(b.scaled) << 25 |
         static_cast<uint32_t>(b.pick) << 26;
}
__device__ inline ModBlock unpack_block(uint32_t v) {
  return ModBlock{static_cast<uint16_t>(v & 0x3ffu), static_cast<uint8_t>((v >> 10) & 0xffu),
                  static_cast<uint8_t>((v >> 18) & 0x3fu), static_cast<uint8_t>((v >> 24) & 1u),
                  static_cast<uint8_t>((v >> 25) & 1u), static_cast<uint8_t>(v >> 26)};
}

struct SplitOperand {
  int64_t lines, line_stride, k_stride, plane, ld;  // strides of X in doubles, ld in bytes
  const double* X;
  const int32_t* E;
  int8_t* D;
  int tiles, blocks, panels, unused;  // tiles: blocks of threads along the lines
};
struct SplitArgs {
  SplitOperand op[2];  // A, B
  int64_t K, kp;
  int L, gbits;
  uint32_t b[2][kModMaxBlocks];
};

// 32 bits of the integer I starting at bit `lo` (uniform), by unrolled selects.
template <int NW>
__device__ inline uint32_t bits_at(const uint64_t (&I)[NW], int lo) {
  const int wi = lo >> 6, b = lo & 63;
  uint64_t v = word_or_zero<NW>(I, wi) >> b;
  if (b > 32) v |= word_or_zero<NW>(I, wi + 1) << (64 - b);
  return static_cast<uint32_t>(v);
}

__device__ inline uint32_t pack4(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  // the low bytes of a, b, c, d
  const uint32_t ab = __builtin_amdgcn_perm(b, a, 0x0c0c0400u), cd = __builtin_amdgcn_perm(d, c, 0x0c0c0400u);
  return ab | (cd << 16);
}

// The integers of a thread's four elements: 32 bits of each from bit `lo` on.
template <int NW>
struct RegisterWords {
  uint64_t I[4][NW];
  __device__ inline void get(int lo, uint32_t (&v)[4]) const {
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = bits_at<NW>(I[i], lo);
  }
};
// Long integers wait in LDS, [dword][thread] with the four elements side by side,
// instead of unrolled selects over up to 15 words.
struct LdsWords {
  const uint4* w;
  int threads;
  __device__ inline void get(int lo, uint32_t (&v)[4]) const {
    const int wi = lo >> 5, b = lo & 31;
    const uint4 x = w[wi * threads], y = w[(wi + 1) * threads];
    v[0] = __builtin_amdgcn_alignbit(y.x, x.x, b);
    v[1] = __builtin_amdgcn_alignbit(y.y, x.y, b);
    v[2] = __builtin_amdgcn_alignbit(y.z, x.z, b);
    v[3] = __builtin_amdgcn_alignbit(y.w, x.w, b);
  }
};

// The residue panels c0 .. c1 - 1 of one block with at most ND dwords of bits.
template <int ND, class Words>
__device__ inline void residue_panels(const Words& words, const float (&sgn)[4], ModBlock blk, int c0, int c1,
                                      int8_t* __restrict__ out, int64_t kp, bool store) {
  uint32_t e[4][ND];
#pragma unroll
  for (int j = 0; j < ND; ++j) {
    const int left = blk.bits - 32 * j;  // uniform
    const uint32_t mask = left >= 32 ? 0xffffffffu : (left > 0 ? (1u << left) - 1u : 0u);
    uint32_t v[4] = {0, 0, 0, 0};
    if (left > 0) words.get(blk.lo + 32 * j, v);
#pragma unroll
    for (int i = 0; i < 4; ++i) e[i][j] = v[i] & mask;
  }
  const int row = blk.scaled ? mod_row(blk.count, 0) : kModRows;
  for (int c = c0; c < c1; ++c) {
    const uint32_t* t = kResidueTable.row[row + c];
    uint32_t k[ND];
#pragma unroll
    for (int j = 0; j < ND; ++j) k[j] = t[j];
    const float m = __uint_as_float(t[6]), r = __uint_as_float(t[7]);
    uint32_t v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      uint32_t x = 0;
#pragma unroll
      for (int j = 0; j < ND; ++j) x = __builtin_amdgcn_udot4(e[i][j], k[j], x, false);
      const float f = static_cast<float>(x);
      const float q = __builtin_rintf(f * r);
      // integers below 2^24: exact; the low byte of 1.5 2^23 + s is s modulo 256
      v[i] = __float_as_uint(__builtin_fmaf(__builtin_fmaf(-q, m, f), sgn[i], 12582912.0f));
    }
    if (store) *reinterpret_cast<uint32_t*>(out + static_cast<int64_t>(c) * kp) = pack4(v[0], v[1], v[2], v[3]);
  }
}

// The sub-digit panels of one digit: the C balanced sub-digits, then the sums of
// every two of them (each in [-128, 127]); one sub-digit is the digit itself.
template <int C, class Words>
__device__ inline void direct_panels(const Words& words, const float (&sgn)[4], ModBlock blk,
                                     int8_t* __restrict__ out, int64_t kp, bool store) {
  int32_t s[4][C];
  uint32_t f[4];
  words.get(blk.lo, f);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int32_t d = static_cast<int32_t>(f[i] & ((1u << blk.bits) - 1u));
    int32_t v = sgn[i] < 0.0f ? -d : d;
#pragma unroll
    for (int j = 0; j + 1 < C; ++j) {
      s[i][j] = static_cast<int32_t>(static_cast<uint32_t>(v) << 25) >> 25;  // balanced: -64 .. 63
      v = (v - s[i][j]) >> 7;
    }
    s[i][C - 1] = v;
  }
  int p = 0;
  auto put = [&](int32_t a, int32_t b, int32_t c, int32_t d) {
    if (store)
      *reinterpret_cast<uint32_t*>(out + static_cast<int64_t>(p) * kp) =
          pack4(static_cast<uint32_t>(a), static_cast<uint32_t>(b), static_cast<uint32_t>(c),
                static_cast<uint32_t>(d));
    ++p;
  };
#pragma unroll
  for (int j = 0; j < C; ++j) put(s[0][j], s[1][j], s[2][j], s[3][j]);
#pragma unroll
  for (int j = 0; j < C; ++j)
#pragma unroll
    for (int l = j + 1; l < C; ++l)
      put(s[0][j] + s[0][l], s[1][j] + s[1][l], s[2][j] + s[2][l], s[3][j] + s[3][l]);
}

// One sub-digit of a digit (blk.pick - 1; blk.scaled: the top one, which takes the rest).
template <class Words>
__device__ inline void sub_digit_panel(const Words& words, const float (&sgn)[4], ModBlock blk,
                                       int8_t* __restrict__ out, bool store) {
  uint32_t f[4], v[4];
  words.get(blk.lo, f);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int32_t d = static_cast<int32_t>(f[i] & ((1u << blk.bits) - 1u));
    int32_t x = sgn[i] < 0.0f ? -d : d;
    for (int j = 1; j < blk.pick; ++j) x = (x + 64) >> 7;  // (x - balanced(x)) / 128
    if (!blk.scaled) x = static_cast<int32_t>(static_cast<uint32_t>(x) << 25) >> 25;
    v[i] = static_cast<uint32_t>(x);
  }
  if (store) *reinterpret_cast<uint32_t*>(out) = pack4(v[0], v[1], v[2], v[3]);
}

// The panels p0 .. p1 - 1 of the operand, all its blocks in turn.
template <class Words>
__device__ inline void all_panels(const Words& words, const float (&sgn)[4], const uint32_t* __restrict__ blocks,
                                  int count, int p0, int p1, int8_t* __restrict__ out, int64_t kp, bool store) {
  int first = 0;
  for (int b = 0; b < count; ++b) {
    const ModBlock blk = unpack_block(blocks[b]);
    if (blk.residue) {
      const int c0 = p0 > first ? p0 - first : 0, c1 = p1 - first < blk.count ? p1 - first : blk.count;
      if (c0 < c1) {
        if (blk.bits <= 32) residue_panels<1>(words, sgn, blk, c0, c1, out, kp, store);
        else if (blk.bits <= 64) residue_panels<2>(words, sgn, blk, c0, c1, out, kp, store);
        else if (blk.bits <= 128) residue_panels<4>(words, sgn, blk, c0, c1, out, kp, store);
        else residue_panels<6>(words, sgn, blk, c0, c1, out, kp, store);
      }
    } else if (first >= p0 && first < p1) {  // a digit's panels go together
      if (blk.pick) sub_digit_panel(words, sgn, blk, out, store);
      else if (blk.count == 1) direct_panels<1>(words, sgn, blk, out, kp, store);
      else if (blk.count == 3) direct_panels<2>(words, sgn, blk, out, kp, store);
      else if (blk.count == 6) direct_panels<3>(words, sgn, blk, out, kp, store);
      else direct_panels<4>(words, sgn, blk, out, kp, store);
    }
    out += static_cast<int64_t>(blk.count) * kp;
    first += blk.count;
  }
}

// kWin: 2 or 4, the 128- or 256-bit integer floor; 0, the general one.
template <int NW, int ML, int TK, int kWin>
__global__ void __launch_bounds__(4 * TK) modular_split_kernel(SplitArgs) {
  constexpr int kPitch = TK + 2;
  extern __shared__ double tile[];  // [L][kLines][kPitch]
  // the argument in place (see modular_accum.hip)
  const SplitArgs& args = *(const SplitArgs*)__builtin_amdgcn_kernarg_segment_ptr();
  const int which = static_cast<int>(blockIdx.x) < args.op[0].tiles ? 0 : 1;
  const SplitOperand& op = args.op[which];
  const int L = args.L, t = threadIdx.x;
  const int64_t c0 = static_cast<int64_t>(blockIdx.x - (which ? args.op[0].tiles : 0)) * kLines;
  const int64_t k0 = static_cast<int64_t>(blockIdx.y) * TK, K = args.K, kp = args.kp, lines = op.lines;
  // the tile's limbs, 4 elements per thread (+0.0 outside the operand)
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int x = t + i * 4 * TK;
    const bool rows = op.k_stride == 1;
    const int line = rows ? x / TK : x % kLines, kk = rows ? x % TK : x / kLines;
    const bool ok = c0 + line < lines && k0 + kk < K;
    const int64_t idx = ok ? (c0 + line) * op.line_stride + (k0 + kk) * op.k_stride : 0;
    for (int l = 0; l < L; ++l)
      tile[(l * kLines + line) * kPitch + kk] = ok ? op.X[static_cast<int64_t>(l) * op.plane + idx] : 0.0;
  }
  __syncthreads();
  const int line = t / (TK / 4), kq = 4 * (t % (TK / 4));
  const int64_t c = c0 + line, kk = k0 + kq;
  const bool store = c < lines && kk < kp;
  const int g = (c < lines ? op.E[c] : 0) - args.gbits;  // the grid exponent E - w S
  RegisterWords<NW> words;
  float sgn[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    double xs[ML];
#pragma unroll
    for (int l = 0; l < ML; ++l) xs[l] = l < L ? tile[(l * kLines + line) * kPitch + kq + i] : 0.0;
    bool neg;
    if constexpr (kWin == 2)
      neg = floor_on_grid_128<ML>(xs, L, g, words.I[i]);
    else if constexpr (kWin == 4)
      neg = floor_on_grid_256<ML>(xs, L, g, words.I[i]);
    else
      neg = floor_on_grid<NW, ML>(xs, L, g, words.I[i]);
    sgn[i] = neg ? -1.0f : 1.0f;
  }
  int8_t* out = op.D + c * op.ld + kk;
  const int z = blockIdx.z, nz = gridDim.z;
  const int p0 = op.panels * z / nz, p1 = op.panels * (z + 1) / nz;
  if constexpr (NW >= 8) {
    __syncthreads();  // the tile's readers are done
    uint4* w = reinterpret_cast<uint4*>(tile) + t;
#pragma unroll
    for (int i = 0; i < 2 * NW + 1; ++i) {
      auto at = [&](int e) {
        return i < 2 * NW ? static_cast<uint32_t>(words.I[e][i / 2 < NW ? i / 2 : 0] >> (32 * (i & 1))) : 0u;
      };
      w[i * 4 * TK] = make_uint4(at(0), at(1), at(2), at(3));
    }
    // every thread reads its own words only
    all_panels(LdsWords{w, 4 * TK}, sgn, args.b[which], op.blocks, p0, p1, out, kp, store);
  } else {
    all_panels(words, sgn, args.b[which], op.blocks, p0, p1, out, kp, store);
  }
}

template <int NW, int ML, int TK, int kWin>
hipError_t launch_split_tile(SplitArgs& a, hipStream_t stream) {
  size_t lds = sizeof(double) * static_cast<size_t>(a.L) * kLines * (TK + 2);
  if (NW >= 8) lds = std::max(lds, sizeof(uint4) * (2 * NW + 1) * 4 * TK);
  int64_t gx = 0;
  for (SplitOperand& op : a.op) {
    op.tiles = static_cast<int>((op.lines + kLines - 1) / kLines);
    gx += op.tiles;
  }
  const int64_t gy = (a.kp + TK - 1) / TK;
  const int64_t gz = mod_split_shares(gx * gy);
  auto kernel = modular_split_kernel<NW, ML, TK, kWin>;
  if (lds > 64 * 1024) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(gx), static_cast<unsigned>(gy), static_cast<unsigned>(gz)),
                     dim3(4 * TK), lds, stream, a);
  return hipGetLastError();
}

}  // namespace

// Grid limits of the tiles above, whichever is taken: below 2^32 threads along x (blocks
// of up to 512 threads per 16 lines) and 65535 blocks along y (64 values of k at least).
bool modular_split_fits(int64_t m, int64_t n, int64_t k) {
  if (m > (int64_t{1} << 30) || n > (int64_t{1} << 30)) return false;
  return mod_split_tiles(m, n) * 512 < (int64_t{1} << 32) && (mod_kp(k) + 63) / 64 <= 65535;
}

hipError_t launch_modular_split(int64_t m, int64_t n, int64_t k, int L, int S, int w, const double* A,
                                const double* B, const int32_t* EA, const int32_t* EB, int8_t* DA, int8_t* DB,
                                const std::vector<ModBlock>& ba, int pa, const std::vector<ModBlock>& bb, int pb,
                                hipStream_t stream) {
  if (m == 0 || n == 0 || k == 0) return hipSuccess;
  if (ba.size() > static_cast<size_t>(kModMaxBlocks) || bb.size() > static_cast<size_t>(kModMaxBlocks) ||
      !modular_split_fits(m, n, k))
    return hipErrorInvalidValue;
  SplitArgs a{};
  a.K = k;
  a.kp = mod_kp(k);
  a.L = L;
  a.gbits = w * S;
  a.op[0] = SplitOperand{m, k, 1, m * k, pa * a.kp, A, EA, DA, 0, static_cast<int>(ba.size()), pa, 0};
  a.op[1] = SplitOperand{n, 1, n, k * n, pb * a.kp, B, EB, DB, 0, static_cast<int>(bb.size()), pb, 0};
  std::transform(ba.begin(), ba.end(), a.b[0], pack_block);
  std::transform(bb.begin(), bb.end(), a.b[1], pack_block);
  const int bits = w * S, words = (bits + 52 + 63) / 64;
  if (L <= 2 && bits <= 128) return launch_split_tile<2, 2, 128, 2>(a, stream);
  if (L <= 4 && bits <= 256) return launch_split_tile<4, 4, 128, 4>(a, stream);
  if (L <= 4 && words <= 8) return launch_split_tile<8, 4, 64, 0>(a, stream);
  if (L <= 8 && words <= 8) return launch_split_tile<8, 8, 64, 0>(a, stream);
  if (words <= 15) return launch_split_tile<15, 16, 64, 0>(a, stream);
  return hipErrorInvalidValue;
}

}  // namespace mdg
