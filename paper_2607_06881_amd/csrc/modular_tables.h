// Tables of the residue systems (modular.h) for the device, computed at compile
// time from the moduli: for the first N of them, with M their product and
// W_i = M / m_i, the constants of the residues (W_i^-1 mod m_i among them) and
// those of the recovery V = sum_i y_i W_i - q M.
#pragma once

#include <stdint.h>

#include "modular.h"

namespace mdg {

// Row of modulus i of the N-moduli system.
__host__ __device__ constexpr int mod_row(int N, int i) { return N * (N - 1) / 2 + i; }
constexpr int kModRows = kMaxModuli * (kMaxModuli + 1) / 2;

struct ModLimbs {
  uint32_t x[kModLimbs] = {};
};

constexpr void mul_limbs(ModLimbs* v, int f) {
  uint64_t carry = 0;
  for (int j = 0; j < kModLimbs; ++j) {
    const uint64_t p = static_cast<uint64_t>(v->x[j]) * static_cast<uint64_t>(f) + carry;
    v->x[j] = static_cast<uint32_t>(p);
    carry = p >> 32;
  }
}

constexpr int inverse_mod(int a, int m) {
  int r0 = m, r1 = a % m, t0 = 0, t1 = 1;
  while (r1 != 0) {
    const int q = r0 / r1, r2 = r0 - q * r1, t2 = t0 - q * t1;
    r0 = r1;
    r1 = r2;
    t0 = t1;
    t1 = t2;
  }
  return t0 < 0 ? t0 + m : t0;
}

// 32-bit limbs of M for N moduli.
constexpr int mod_limbs(int N) {
  ModLimbs M;
  M.x[0] = 1;
  for (int i = 0; i < N; ++i) mul_limbs(&M, kModuli[i]);
  int n = 0;
  for (int j = 0; j < kModLimbs; ++j)
    if (M.x[j] != 0) n = j + 1;
  return n;
}

// Residue constants of modulus i scaled by W_i^-1 (row mod_row(N, i)) and unscaled
// (row kModRows + i): six dwords of bytes 256^j f mod m, then m and 1 / m as floats.
struct ResidueTable {
  uint32_t row[kModRows + kMaxModuli][8] = {};
};

constexpr void residue_row(uint32_t (&o)[8], int f, int m) {
  uint32_t c = static_cast<uint32_t>(f % m);
  for (int j = 0; j < 6; ++j) {
    o[j] = 0;
    for (int y = 0; y < 4; ++y) {
      o[j] |= c << (8 * y);
      c = (c << 8) % static_cast<uint32_t>(m);
    }
  }
  o[6] = __builtin_bit_cast(uint32_t, static_cast<float>(m));
  o[7] = __builtin_bit_cast(uint32_t, 1.0f / static_cast<float>(m));
}

constexpr ResidueTable make_residue_table() {
  ResidueTable t;
  for (int N = 1; N <= kMaxModuli; ++N) {
    residue_row(t.row[kModRows + N - 1], 1, kModuli[N - 1]);
    for (int i = 0; i < N; ++i) {
      int prod = 1;  // W_i mod m_i
      for (int j = 0; j < N; ++j)
        if (j != i) prod = prod * (kModuli[j] % kModuli[i]) % kModuli[i];
      residue_row(t.row[mod_row(N, i)], inverse_mod(prod, kModuli[i]), kModuli[i]);
    }
  }
  return t;
}

// The recovery takes the y_i of a system four at a time (a quad) and sixteen
// together: the quads of N moduli, rounded up to fours.
__host__ __device__ constexpr int mod_quads_of(int N) { return (N + 15) / 16 * 4; }

// First row of the N-moduli system: mod_limbs(n) + 1 rows of quads for every n < N.
constexpr int mod_quad_base(int N) {
  int b = 0;
  for (int n = 1; n < N; ++n) b += mod_quads_of(n) * (mod_limbs(n) + 1);
  return b;
}
constexpr int kModQuadRows = mod_quad_base(kMaxModuli + 1);

// Recovery constants: for limb l of the N-moduli system, row mod_quad_base(N) + l
// mod_quads_of(N) + quad holds, for byte c of the limb, the bytes of the quad's four
// W_i in one dword; the rows after the last limb hold the three bytes of
// round(2^24 / m_i).  M: the limbs of M.
struct QuadTable {
  uint32_t row[kModQuadRows][4] = {};
  uint32_t M[kMaxModuli + 1][kModLimbs] = {};
};

constexpr QuadTable make_quad_table() {
  QuadTable t;
  int base = 0;
  ModLimbs W[kMaxModuli];
  ModLimbs M;
  M.x[0] = 1;
  for (int N = 1; N <= kMaxModuli; ++N) {
    const int mN = kModuli[N - 1];
    for (int i = 0; i + 1 < N; ++i) mul_limbs(&W[i], mN);
    W[N - 1] = M;
    mul_limbs(&M, mN);
    int limbs = 0;
    for (int j = 0; j < kModLimbs; ++j) {
      t.M[N][j] = M.x[j];
      if (M.x[j] != 0) limbs = j + 1;
    }
    const int quads = mod_quads_of(N);
    for (int i = 0; i < N; ++i) {
      const uint32_t r = ((uint32_t{1} << 25) / static_cast<uint32_t>(kModuli[i]) + 1) / 2;
      for (int c = 0; c < 4; ++c) {
        for (int j = 0; j < limbs; ++j)
          t.row[base + j * quads + i / 4][c] |= ((W[i].x[j] >> (8 * c)) & 0xffu) << (8 * (i % 4));
        t.row[base + limbs * quads + i / 4][c] |= ((r >> (8 * c)) & 0xffu) << (8 * (i % 4));
      }
    }
    base += quads * (limbs + 1);
  }
  return t;
}

}  // namespace mdg
