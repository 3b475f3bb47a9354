// Steps a4 and a5 from the int8 products of modular.h: every group's value V is
// recovered and added into the exact sum N = sum_t G_t 2^(w (T - t)) of the
// element, which is then rounded as in accum_renorm.hip.
//
// Planes hold four rows per dword (or per 16 bytes, int32): two neighbouring
// threads take two rows each of the four rows of one column, so that a load
// serves both.  (Four elements per thread needed up to 186 registers: two waves per
// SIMD instead of four.)
//
// Residue groups: V = sum_i y_i W_i - q M with q = round(sum_i y_i / m_i)
// (|V| / M < 0.497; the sum in units of 2^-24 is off by less than 0.0004).  The
// bytes of four channels of an element are put into one dword (a byte
// transposition) and multiplied with byte columns of the W_i by v_dot4_u32_u8,
// four products per instruction at the full vector rate, sixteen channels at a
// time, into one 64-bit sum per 32-bit limb; carries are resolved once at the end.
// Every group's rectangles reach the cutoff, so its weight is 1.
//
// Direct groups: V = sum of coef * plane over the sub-digit products (Karatsuba's
// identity) in int64, and the carry chain of the levels.
//
// Bound by integer issue next to the planes' HBM traffic.  Before this form: FP64
// multiply-adds on 32-bit limbs, 5.98 ms for td 8192 x 8192 (93 planes) and 0.83 ms
// for dd 4096 x 4096 (60 planes).
#include <algorithm>
#include <type_traits>
#include <utility>
#include <vector>

#include "digits.h"
#include "internal.h"
#include "modular.h"
#include "modular_tables.h"

namespace mdg {
namespace {

__constant__ const QuadTable kQuadTable = make_quad_table();

constexpr int kElems = 2;        // elements per thread
constexpr int kDirectBatch = 6;  // direct planes loaded together

// The tables are whole dwords, 4-byte aligned: scalar loads ignore the two low bits
// of their base, which the compiler lets point between the fields of a structure of
// bytes and halves.
//
// sixteen channels of a residue group: planes out .. out + channels - 1
struct Block {
  uint32_t where;  // out | table << 16: first plane, row of kQuadTable of limb 0
  uint32_t what;   // channels | limbs << 8 | rows from limb to limb << 16 |
                   // (moduli of the group in its last block, else 0) << 24
};
// one plane of a direct group: value += coef 2^shift plane, of weight 2^(w column)
struct Direct {
  uint32_t where;  // out | column << 16 | shift << 24
  int32_t coef;
};
struct AccumArgs {
  int64_t m, n;
  const uint32_t* P;
  const int32_t *EA, *EB;
  double* C;
  int L, w, base;  // base: the grid scale of N is 2^(EA + EB - base)
  int blocks, directs, columns;  // columns: levels of the carry chain
  Block block[kModMaxChannelBlocks];
  Direct direct[kModMaxDirect];
};
static_assert(sizeof(AccumArgs) <= 4096, "the kernel arguments of one launch");

// The bytes of (a, b, c, d) for this thread's two rows: o[e] holds byte 2 half + e of
// each; sel picks them from two dwords at a time.
__device__ inline void transpose2(uint32_t a, uint32_t b, uint32_t c, uint32_t d, uint32_t sel,
                                  uint32_t (&o)[kElems]) {
  const uint32_t ab = __builtin_amdgcn_perm(b, a, sel), cd = __builtin_amdgcn_perm(d, c, sel);
  o[0] = __builtin_amdgcn_perm(cd, ab, 0x05040100u);
  o[1] = __builtin_amdgcn_perm(cd, ab, 0x07060302u);
}

// N += the residue groups.
template <int NW>
__device__ inline void add_residues(uint64_t (&N)[kElems][NW], const AccumArgs& args,
                                    const uint32_t* __restrict__ p, int64_t unit, uint32_t sel) {
  int64_t acc[2 * NW][kElems];
#pragma unroll
  for (int l = 0; l < 2 * NW; ++l)
#pragma unroll
    for (int e = 0; e < kElems; ++e) acc[l][e] = 0;
  uint32_t f[kElems][3] = {};
  uint32_t next[16];
  auto load = [&](int b) {
    const uint32_t* src = p + (args.block[b].where & 0xffffu) * unit;
    const uint32_t channels = args.block[b].what & 0xffu;
#pragma unroll
    for (uint32_t c = 0; c < 16; ++c) {
      next[c] = 0;
      if (c < channels) next[c] = *src;
      src += unit;
    }
  };
  load(0);
  for (int b = 0; b < args.blocks; ++b) {
    const uint32_t table = args.block[b].where >> 16, what = args.block[b].what;
    const int limbs = (what >> 8) & 0xffu, stride = (what >> 16) & 0xffu, last = what >> 24;
    uint32_t y[4][kElems];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      transpose2(next[4 * u], next[4 * u + 1], next[4 * u + 2], next[4 * u + 3], sel, y[u]);
    if (b + 1 < args.blocks) load(b + 1);
    const uint32_t(*k)[4] = kQuadTable.row + table;
#pragma unroll
    for (int l = 0; l < 2 * NW && l < kModLimbs; ++l) {
      if (l < limbs) {
        uint32_t s[kElems][4] = {};
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int e = 0; e < kElems; ++e)
#pragma unroll
            for (int c = 0; c < 4; ++c) s[e][c] = __builtin_amdgcn_udot4(y[u][e], k[u][c], s[e][c], false);
#pragma unroll
        for (int e = 0; e < kElems; ++e) {
          // columns below 2^20: pairs below 2^32
          const uint32_t lo = s[e][0] + (s[e][1] << 8), hi = s[e][2] + (s[e][3] << 8);
          acc[l][e] += static_cast<int64_t>(static_cast<uint64_t>(hi) * 65536u + lo);
        }
      }
      k += stride;
    }
    k = kQuadTable.row + table + limbs * stride;
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int e = 0; e < kElems; ++e)
#pragma unroll
        for (int c = 0; c < 3; ++c) f[e][c] = __builtin_amdgcn_udot4(y[u][e], k[u][c], f[e][c], false);
    if (last) {
#pragma unroll
      for (int e = 0; e < kElems; ++e) {
        const uint32_t q = (f[e][0] + (f[e][1] << 8) + (f[e][2] << 16) + (1u << 23)) >> 24;
        f[e][0] = f[e][1] = f[e][2] = 0;
#pragma unroll
        for (int l = 0; l < 2 * NW && l < kModLimbs; ++l)
          acc[l][e] -= static_cast<int64_t>(static_cast<uint64_t>(q) * kQuadTable.M[last][l]);
      }
    }
  }
#pragma unroll
  for (int e = 0; e < kElems; ++e) {
    int64_t carry = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      const int64_t x0 = acc[2 * i][e] + carry + static_cast<int64_t>(N[e][i] & 0xffffffffull);
      const int64_t x1 = acc[2 * i + 1][e] + (x0 >> 32) + static_cast<int64_t>(N[e][i] >> 32);
      N[e][i] = (static_cast<uint64_t>(x0) & 0xffffffffull) | (static_cast<uint64_t>(x1) << 32);
      carry = x1 >> 32;
    }
  }
}

template <int NW, bool kResidues>
__global__ void __launch_bounds__(256) modular_accum_kernel(AccumArgs) {
  // the one argument, read in place: as a by-value parameter its indexed tables were
  // copied to scratch memory
  const AccumArgs& args = *(const AccumArgs*)__builtin_amdgcn_kernarg_segment_ptr();
  const int64_t m = args.m, n = args.n;
  const int L = args.L, w = args.w, base = args.base;
  const uint32_t* __restrict__ P = args.P;
  const int32_t* __restrict__ EA = args.EA;
  const int32_t* __restrict__ EB = args.EB;
  double* __restrict__ C = args.C;
  const int64_t j = static_cast<int64_t>(blockIdx.x) * (blockDim.x / 2) + (threadIdx.x >> 1);
  if (j >= n) return;
  const int half = threadIdx.x & 1;
  const uint32_t sel = half ? 0x07030602u : 0x05010400u;
  const int64_t quads = (m + 3) / 4, unit = quads * n, plane = m * n;
  const int ebj = EB[j];
  for (int64_t qi = blockIdx.y; qi < quads; qi += gridDim.y) {
    const uint32_t* p = P + qi * n + j;
    uint64_t N[kElems][NW];
#pragma unroll
    for (int e = 0; e < kElems; ++e)
#pragma unroll
      for (int i = 0; i < NW; ++i) N[e][i] = 0;
    if (args.columns > 0) {
      const uint64_t mask = (1ull << w) - 1ull;
      CarryChain<NW> chain[kElems];
      int64_t v[kElems] = {};
      int col = 0;
      auto step = [&] {
#pragma unroll
        for (int e = 0; e < kElems; ++e) {
          chain[e].step(N[e], v[e], w, mask);
          v[e] = 0;
        }
        ++col;
      };
      for (int d0 = 0; d0 < args.directs; d0 += kDirectBatch) {
        int2 x[kDirectBatch];
#pragma unroll
        for (int u = 0; u < kDirectBatch; ++u)
          x[u] = reinterpret_cast<const int2*>(
              P + (args.direct[d0 + u < args.directs ? d0 + u : 0].where & 0xffffu) * unit)[2 * (qi * n + j) + half];
#pragma unroll
        for (int u = 0; u < kDirectBatch; ++u) {
          if (d0 + u >= args.directs) break;
          const uint32_t where = args.direct[d0 + u].where;
          const int64_t coef = args.direct[d0 + u].coef;
          while (col < static_cast<int>((where >> 16) & 0xffu)) step();
          v[0] += (coef * x[u].x) << (where >> 24);
          v[1] += (coef * x[u].y) << (where >> 24);
        }
      }
      step();  // the last column
#pragma unroll
      for (int e = 0; e < kElems; ++e) chain[e].finish(N[e], w, args.columns - 1);
    }
    if constexpr (kResidues) add_residues<NW>(N, args, p, unit, sel);
#pragma unroll
    for (int e = 0; e < kElems; ++e) {
      const int64_t i = 4 * qi + 2 * half + e;
      if (i < m) round_limbs<NW>(N[e], L, EA[i] + ebj - base, C, plane, i * n + j);
    }
  }
}

// Karatsuba's identity on c sub-digits of 7 bits: the products of the sub-digits
// D_i and of their sums S_ij give sum_i D_i 2^(14 i) + sum_{i<j} (S_ij - D_i - D_j) 2^(7 (i + j)).
void direct_coefs(int w, int64_t (&d)[kDirectTypes]) {
  const int c = w <= 7 ? 1 : (w + 7) / 7;
  int next = c;
  for (int i = 0; i < c; ++i) d[i] += int64_t{1} << (14 * i);
  for (int i = 0; i < c; ++i)
    for (int j = i + 1; j < c; ++j) {
      d[next++] = int64_t{1} << (7 * (i + j));
      d[i] -= int64_t{1} << (7 * (i + j));
      d[j] -= int64_t{1} << (7 * (i + j));
    }
}

// The kernel's view of a plan; false when its planes do not fit the tables.
bool accum_args(const ModPlan& pl, int w, AccumArgs* a) {
  static const std::vector<std::pair<int, int>> systems = [] {
    std::vector<std::pair<int, int>> v;  // limbs and first table row of every system
    for (int i = 0; i <= kMaxModuli; ++i) v.emplace_back(mod_limbs(i), mod_quad_base(i));
    return v;
  }();
  int64_t coef[kDirectTypes] = {};
  direct_coefs(w, coef);
  std::vector<ModGroup> res;
  std::vector<Direct> dir;
  for (const ModGroup& g : pl.groups) {
    if (g.residue) {
      res.push_back(g);
      continue;
    }
    for (int i = 0; i < g.count; ++i) {
      int64_t c = coef[i];
      int shift = 0;
      while (c != static_cast<int32_t>(c)) {  // the large ones are multiples of 2^21
        if (c & 1) return false;
        c >>= 1;
        ++shift;
      }
      if (g.shift / w > 255) return false;
      dir.push_back(Direct{static_cast<uint32_t>(g.out + 4 * i) | static_cast<uint32_t>(g.shift / w) << 16 |
                               static_cast<uint32_t>(shift) << 24,
                           static_cast<int32_t>(c)});
    }
  }
  if (dir.size() > static_cast<size_t>(kModMaxDirect)) return false;
  auto column = [](const Direct& d) { return static_cast<int>((d.where >> 16) & 0xffu); };
  std::stable_sort(dir.begin(), dir.end(), [&](const Direct& x, const Direct& y) { return column(x) < column(y); });
  a->directs = static_cast<int>(dir.size());
  a->columns = dir.empty() ? 0 : column(dir.back()) + 1;
  std::copy(dir.begin(), dir.end(), a->direct);
  for (const ModGroup& g : res) {
    if (g.shift != 0) return false;
    for (int i = 0; i < g.count; i += 16) {
      if (a->blocks == kModMaxChannelBlocks) return false;
      Block& d = a->block[a->blocks++];
      const uint32_t channels = static_cast<uint32_t>(std::min(16, g.count - i));
      d.where = static_cast<uint32_t>(g.out + i) | static_cast<uint32_t>(systems[g.count].second + i / 4) << 16;
      d.what = channels | static_cast<uint32_t>(systems[g.count].first) << 8 |
               static_cast<uint32_t>(mod_quads_of(g.count)) << 16 |
               static_cast<uint32_t>(i + 16 >= g.count ? g.count : 0) << 24;
    }
  }
  return true;
}

}  // namespace

bool modular_accum_fits(const ModPlan& pl, int w) {
  AccumArgs a{};
  return accum_args(pl, w, &a);
}

hipError_t launch_modular_accum(int64_t m, int64_t n, int L, int T, int w, const ModPlan& pl, const uint32_t* P,
                                const int32_t* EA, const int32_t* EB, double* C, hipStream_t stream) {
  if (m == 0 || n == 0) return hipSuccess;
  AccumArgs a{};
  if (!accum_args(pl, w, &a)) return hipErrorInvalidValue;
  const int64_t quads = mod_quads(m);
  const dim3 grid(static_cast<unsigned>((n + 127) / 128), static_cast<unsigned>(quads < 65535 ? quads : 65535));
  a.m = m;
  a.n = n;
  a.P = P;
  a.EA = EA;
  a.EB = EB;
  a.C = C;
  a.L = L;
  a.w = w;
  a.base = 2 * w + w * T;
  const int words = accum_words(T + 1, w);
  auto go = [&](auto nw) {
    constexpr int NW = decltype(nw)::value;
    if (a.blocks)
      hipLaunchKernelGGL((modular_accum_kernel<NW, true>), grid, dim3(256), 0, stream, a);
    else
      hipLaunchKernelGGL((modular_accum_kernel<NW, false>), grid, dim3(256), 0, stream, a);
    return hipGetLastError();
  };
  if (words <= 2) return go(std::integral_constant<int, 2>{});
  if (words <= 3) return go(std::integral_constant<int, 3>{});
  if (words <= 4) return go(std::integral_constant<int, 4>{});
  if (words <= 5) return go(std::integral_constant<int, 5>{});
  if (words <= 8) return go(std::integral_constant<int, 8>{});
  if (words <= kModMaxWords) return go(std::integral_constant<int, kModMaxWords>{});
  return hipErrorInvalidValue;
}

}  // namespace mdg
