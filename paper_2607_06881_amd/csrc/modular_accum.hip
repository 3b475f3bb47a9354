// Steps a4 and a5 from the int8 products of modular.h: every group's value V is
// recovered and added into the exact sum N = sum_t G_t 2^(w (T - t)) of the
// element, which is then rounded as in accum_renorm.hip.
//
// Planes hold four rows per dword (or per 16 bytes, int32): a thread takes four
// consecutive rows of one column, so its four elements come in one load per
// plane.  Residue groups: V = sum_i y_i W_i - q M with q = rint(sum_i y_i / m_i)
// (|V| / M < 0.497, so the fraction is far from a tie), formed in 32-bit limbs by
// FP64 multiply-adds: y_i < 2^8, limbs below 2^32 and at most 40 terms keep every
// sum an integer below 2^46.  FP64 multiply-adds run at the full vector rate here,
// four times that of 32 x 32-bit integer multiply-adds with 64-bit sums.  Direct
// groups: V = sum of coef * plane over the sub-digit products (Karatsuba's
// identity), in int64.
#include <type_traits>

#include "digits.h"
#include "internal.h"
#include "modular.h"
#include "modular_tables.h"

namespace mdg {
namespace {

constexpr int kChunk = 4;  // limbs formed together

struct AccumGroups {
  int count;
  ModGroup g[kModMaxGroups];
};
struct DirectCoefs {
  int64_t c[kDirectTypes];
};

// N += V 2^sh modulo 2^(64 NW), V a two's-complement integer of three words.
template <int NW>
__device__ inline void add_words(uint64_t (&N)[NW], uint64_t v0, uint64_t v1, int64_t v2, int sh) {
  const int w = sh >> 6, b = sh & 63;
  const uint64_t ext = static_cast<uint64_t>(v2 >> 63), u2 = static_cast<uint64_t>(v2);
  const uint64_t t0 = v0 << b;
  const uint64_t t1 = b ? (v1 << b) | (v0 >> (64 - b)) : v1;
  const uint64_t t2 = b ? (u2 << b) | (v1 >> (64 - b)) : u2;
  const uint64_t t3 = b ? (ext << b) | (u2 >> (64 - b)) : ext;
  uint64_t carry = 0;
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    const uint64_t t = i < w ? 0ull : (i == w ? t0 : (i == w + 1 ? t1 : (i == w + 2 ? t2 : (i == w + 3 ? t3 : ext))));
    const uint64_t s = N[i] + t;
    const uint64_t c1 = s < t;
    const uint64_t s2 = s + carry;
    const uint64_t c2 = s2 < s;
    N[i] = s2;
    carry = c1 | c2;
  }
}

// The integer value of a double, |x| < 2^51.
__device__ inline int64_t to_int(double x) {
  return __double_as_longlong(x + 6755399441055744.0) - __double_as_longlong(6755399441055744.0);
}

template <int NW>
__global__ void __launch_bounds__(256) modular_accum_kernel(int64_t m, int64_t n, int L, int base,
                                                            const uint32_t* __restrict__ P,
                                                            const int32_t* __restrict__ EA,
                                                            const int32_t* __restrict__ EB, double* __restrict__ C,
                                                            AccumGroups groups, DirectCoefs coefs) {
  const int64_t j = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (j >= n) return;
  const int64_t quads = (m + 3) / 4, unit = quads * n, plane = m * n;
  const int ebj = EB[j];
  for (int64_t qi = blockIdx.y; qi < quads; qi += gridDim.y) {
    const uint32_t* p = P + qi * n + j;
    uint64_t N[4][NW];
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int i = 0; i < NW; ++i) N[e][i] = 0;
    for (int gi = 0; gi < groups.count; ++gi) {
      const ModGroup g = groups.g[gi];
      if (g.residue) {
        const uint32_t* y = p + g.out * unit;
        const int row = mod_row(g.count, 0);
        double q[4] = {0.0, 0.0, 0.0, 0.0};
        const int chunks = kModTables.chunks[g.count];
        for (int c = 0; c < chunks; ++c) {
          double s[4][kChunk];
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int l = 0; l < kChunk; ++l) s[e][l] = 0.0;
          for (int i0 = 0; i0 < g.count; i0 += 8) {
            uint32_t v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = y[static_cast<int64_t>(i0 + u < g.count ? i0 + u : 0) * unit];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
              if (i0 + u >= g.count) break;
              const double* W = kModTables.W[row + i0 + u] + c * kChunk;
              const double r = kModTables.r[i0 + u];
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                const double d = static_cast<double>((v[u] >> (8 * e)) & 0xffu);
#pragma unroll
                for (int l = 0; l < kChunk; ++l)
                  s[e][l] = __builtin_fma(d, W[l], s[e][l]);
                if (c == 0) q[e] = __builtin_fma(d, r, q[e]);
              }
            }
          }
          const double* M = kModTables.M[g.count] + c * kChunk;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            if (c == 0) q[e] = __builtin_rint(q[e]);
            int64_t x[kChunk];
#pragma unroll
            for (int l = 0; l < kChunk; ++l)
              x[l] = to_int(__builtin_fma(-q[e], M[l], s[e][l]));
            x[1] += x[0] >> 32;
            x[2] += x[1] >> 32;
            x[3] += x[2] >> 32;
            const uint64_t lo = 0xffffffffull;
            add_words<NW>(N[e], (static_cast<uint64_t>(x[0]) & lo) | (static_cast<uint64_t>(x[1]) << 32),
                          (static_cast<uint64_t>(x[2]) & lo) | (static_cast<uint64_t>(x[3]) << 32), x[3] >> 32,
                          g.shift + 128 * c);
          }
        }
      } else {
        const int4* y = reinterpret_cast<const int4*>(P + g.out * unit) + qi * n + j;
        int64_t v[4] = {0, 0, 0, 0};
        for (int i = 0; i < g.count; ++i) {
          const int4 d = y[static_cast<int64_t>(i) * unit];
          const int64_t f = coefs.c[i];
          v[0] += f * d.x;
          v[1] += f * d.y;
          v[2] += f * d.z;
          v[3] += f * d.w;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) add_shifted_signed<NW>(N[e], v[e], g.shift);
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int64_t i = 4 * qi + e;
      if (i < m) round_limbs<NW>(N[e], L, EA[i] + ebj - base, C, plane, i * n + j);
    }
  }
}

// Karatsuba's identity on c sub-digits of 7 bits: the products of the sub-digits
// D_i and of their sums S_ij give sum_i D_i 2^(14 i) + sum_{i<j} (S_ij - D_i - D_j) 2^(7 (i + j)).
DirectCoefs direct_coefs(int w) {
  DirectCoefs d{};
  const int c = w <= 7 ? 1 : (w + 7) / 7;
  int next = c;
  for (int i = 0; i < c; ++i) d.c[i] += int64_t{1} << (14 * i);
  for (int i = 0; i < c; ++i)
    for (int j = i + 1; j < c; ++j) {
      d.c[next++] = int64_t{1} << (7 * (i + j));
      d.c[i] -= int64_t{1} << (7 * (i + j));
      d.c[j] -= int64_t{1} << (7 * (i + j));
    }
  return d;
}

}  // namespace

hipError_t launch_modular_accum(int64_t m, int64_t n, int L, int T, int w, const ModPlan& pl, const uint32_t* P,
                                const int32_t* EA, const int32_t* EB, double* C, hipStream_t stream) {
  if (m == 0 || n == 0) return hipSuccess;
  if (pl.groups.size() > static_cast<size_t>(kModMaxGroups)) return hipErrorInvalidValue;
  AccumGroups ag;
  ag.count = static_cast<int>(pl.groups.size());
  std::copy(pl.groups.begin(), pl.groups.end(), ag.g);
  const DirectCoefs dc = direct_coefs(w);
  const int64_t quads = mod_quads(m);
  const dim3 grid(static_cast<unsigned>((n + 255) / 256), static_cast<unsigned>(quads < 65535 ? quads : 65535));
  const int base = 2 * w + w * T, words = accum_words(T + 1, w);
  auto go = [&](auto nw) {
    hipLaunchKernelGGL((modular_accum_kernel<decltype(nw)::value>), grid, dim3(256), 0, stream, m, n, L, base, P, EA,
                       EB, C, ag, dc);
    return hipGetLastError();
  };
  if (words <= 2) return go(std::integral_constant<int, 2>{});
  if (words <= 3) return go(std::integral_constant<int, 3>{});
  if (words <= 4) return go(std::integral_constant<int, 4>{});
  if (words <= 5) return go(std::integral_constant<int, 5>{});
  if (words <= 7) return go(std::integral_constant<int, 7>{});
  if (words <= 10) return go(std::integral_constant<int, 10>{});
  if (words <= kModMaxWords) return go(std::integral_constant<int, kModMaxWords>{});
  return hipErrorInvalidValue;
}

}  // namespace mdg
