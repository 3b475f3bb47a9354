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
#include <algorithm>

#include "digits.h"
#include "internal.h"
#include "modular.h"
#include "modular_tables.h"

namespace mdg {
namespace {

constexpr int kLines = 16;

__constant__ const ResidueTable kResidueTable = make_residue_table();

// The blocks in one dword each (scalar loads need whole, aligned dwords).
struct SplitBlocks {
  int count;
  uint32_t b[kModMaxBlocks];
};
inline uint32_t pack_block(const ModBlock& b) {
  return b.lo | static_cast<uint32_t>(b.bits) << 10 | static_cast<uint32_t>(b.count) << 18 |
         static_cast<uint32_t>(b.residue) << 24 | static_cast<uint32_t>(b.scaled) << 25;
}
__device__ inline ModBlock unpack_block(uint32_t v) {
  return ModBlock{static_cast<uint16_t>(v & 0x3ffu), static_cast<uint8_t>((v >> 10) & 0xffu),
                  static_cast<uint8_t>((v >> 18) & 0x3fu), static_cast<uint8_t>((v >> 24) & 1u),
                  static_cast<uint8_t>((v >> 25) & 1u)};
}

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

// The residue panels of one block with at most ND dwords of bits.
template <int NW, int ND>
__device__ inline void residue_panels(const uint64_t (&I)[4][NW], const float (&sgn)[4], ModBlock blk,
                                      int8_t* __restrict__ out, int64_t kp, bool store) {
  uint32_t e[4][ND];
#pragma unroll
  for (int j = 0; j < ND; ++j) {
    const int left = blk.bits - 32 * j;  // uniform
    const uint32_t mask = left >= 32 ? 0xffffffffu : (left > 0 ? (1u << left) - 1u : 0u);
#pragma unroll
    for (int i = 0; i < 4; ++i) e[i][j] = left > 0 ? bits_at<NW>(I[i], blk.lo + 32 * j) & mask : 0u;
  }
  const int row = blk.scaled ? mod_row(blk.count, 0) : kModRows;
  for (int c = 0; c < blk.count; ++c) {
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
template <int NW, int C>
__device__ inline void direct_panels(const uint64_t (&I)[4][NW], const float (&sgn)[4], ModBlock blk,
                                     int8_t* __restrict__ out, int64_t kp, bool store) {
  int32_t s[4][C];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int32_t d = static_cast<int32_t>(bits_at<NW>(I[i], blk.lo) & ((1u << blk.bits) - 1u));
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

// kWin: 2 or 4, the 128- or 256-bit integer floor; 0, the general one.
template <int NW, int ML, int TK, int kWin>
__global__ void __launch_bounds__(4 * TK) modular_split_kernel(int64_t lines, int64_t K, int64_t line_stride,
                                                               int64_t k_stride, int64_t plane, int64_t kp,
                                                               int64_t ld, int L, int gbits,
                                                               const double* __restrict__ X,
                                                               const int32_t* __restrict__ E,
                                                               int8_t* __restrict__ D, SplitBlocks blocks) {
  constexpr int kPitch = TK + 2;
  extern __shared__ double tile[];  // [L][kLines][kPitch]
  const int t = threadIdx.x;
  const int64_t c0 = static_cast<int64_t>(blockIdx.x) * kLines;
  const int64_t k0 = static_cast<int64_t>(blockIdx.y) * TK;
  // the tile's limbs, 4 elements per thread (+0.0 outside the operand)
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int x = t + i * 4 * TK;
    int line, kk;
    if (k_stride == 1) {
      line = x / TK;
      kk = x % TK;
    } else {
      line = x % kLines;
      kk = x / kLines;
    }
    const bool ok = c0 + line < lines && k0 + kk < K;
    const int64_t idx = ok ? (c0 + line) * line_stride + (k0 + kk) * k_stride : 0;
    for (int l = 0; l < L; ++l)
      tile[(l * kLines + line) * kPitch + kk] = ok ? X[static_cast<int64_t>(l) * plane + idx] : 0.0;
  }
  __syncthreads();
  const int line = t / (TK / 4), kq = 4 * (t % (TK / 4));
  const int64_t c = c0 + line, kk = k0 + kq;
  const bool store = c < lines && kk < kp;
  const int g = (c < lines ? E[c] : 0) - gbits;  // the grid exponent E - w S
  uint64_t I[4][NW];
  float sgn[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    double xs[ML];
#pragma unroll
    for (int l = 0; l < ML; ++l) xs[l] = l < L ? tile[(l * kLines + line) * kPitch + kq + i] : 0.0;
    bool neg;
    if constexpr (kWin == 2)
      neg = floor_on_grid_128<ML>(xs, L, g, I[i]);
    else if constexpr (kWin == 4)
      neg = floor_on_grid_256<ML>(xs, L, g, I[i]);
    else
      neg = floor_on_grid<NW, ML>(xs, L, g, I[i]);
    sgn[i] = neg ? -1.0f : 1.0f;
  }
  int8_t* out = D + c * ld + kk;
  for (int b = 0; b < blocks.count; ++b) {
    const ModBlock blk = unpack_block(blocks.b[b]);
    if (blk.residue) {
      if (blk.bits <= 32) residue_panels<NW, 1>(I, sgn, blk, out, kp, store);
      else if (blk.bits <= 64) residue_panels<NW, 2>(I, sgn, blk, out, kp, store);
      else if (blk.bits <= 128) residue_panels<NW, 4>(I, sgn, blk, out, kp, store);
      else residue_panels<NW, 6>(I, sgn, blk, out, kp, store);
    } else if (blk.count == 1) {
      direct_panels<NW, 1>(I, sgn, blk, out, kp, store);
    } else if (blk.count == 3) {
      direct_panels<NW, 2>(I, sgn, blk, out, kp, store);
    } else if (blk.count == 6) {
      direct_panels<NW, 3>(I, sgn, blk, out, kp, store);
    } else {
      direct_panels<NW, 4>(I, sgn, blk, out, kp, store);
    }
    out += static_cast<int64_t>(blk.count) * kp;
  }
}

template <int NW, int ML, int TK, int kWin>
hipError_t launch_split_tile(int64_t lines, int64_t K, int64_t ls, int64_t ks, int64_t plane, int64_t kp, int L,
                             int gbits, const double* X, const int32_t* E, int8_t* D,
                             const std::vector<ModBlock>& blocks, int panels, hipStream_t stream) {
  if (blocks.size() > static_cast<size_t>(kModMaxBlocks) || panels > kModMaxPanels) return hipErrorInvalidValue;
  SplitBlocks sb;
  sb.count = static_cast<int>(blocks.size());
  std::transform(blocks.begin(), blocks.end(), sb.b, pack_block);
  const size_t lds = sizeof(double) * static_cast<size_t>(L) * kLines * (TK + 2);
  const int64_t gx = (lines + kLines - 1) / kLines, gy = (kp + TK - 1) / TK;
  if (gy > 65535 || gx > 0x7fffffff) return hipErrorInvalidValue;
  auto kernel = modular_split_kernel<NW, ML, TK, kWin>;
  if (lds > 64 * 1024) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(gx), static_cast<unsigned>(gy)), dim3(4 * TK), lds, stream,
                     lines, K, ls, ks, plane, kp, static_cast<int64_t>(panels) * kp, L, gbits, X, E, D, sb);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_modular_split(int64_t rows, int64_t cols, int L, int S, int w, int axis, const double* X,
                                const int32_t* E, int8_t* D, const ModPlan& pl, hipStream_t stream) {
  const int64_t lines = axis == 0 ? rows : cols, K = axis == 0 ? cols : rows;
  if (lines == 0 || K == 0) return hipSuccess;
  const int64_t ls = axis == 0 ? cols : 1, ks = axis == 0 ? 1 : cols, plane = rows * cols, kp = mod_kp(K);
  const std::vector<ModBlock>& blocks = axis == 0 ? pl.a : pl.b;
  const int panels = axis == 0 ? pl.pa : pl.pb, bits = w * S, words = (bits + 52 + 63) / 64;
#define MDG_MOD_SPLIT(NW, ML, TK, WIN) \
  launch_split_tile<NW, ML, TK, WIN>(lines, K, ls, ks, plane, kp, L, bits, X, E, D, blocks, panels, stream)
  if (L <= 2 && bits <= 128) return MDG_MOD_SPLIT(2, 2, 128, 2);
  if (L <= 4 && bits <= 256) return MDG_MOD_SPLIT(4, 4, 128, 4);
  if (L <= 4 && words <= 8) return MDG_MOD_SPLIT(8, 4, 128, 0);
  if (L <= 8 && words <= 8) return MDG_MOD_SPLIT(8, 8, 64, 0);
  if (words <= 15) return MDG_MOD_SPLIT(15, 16, 64, 0);
#undef MDG_MOD_SPLIT
  return hipErrorInvalidValue;
}

}  // namespace mdg
