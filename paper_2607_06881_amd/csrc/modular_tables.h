// Tables of the residue systems (modular.h) for the device: for the first N
// moduli, M = their product, W_i = M / m_i and W_i^-1 mod m_i, and the constants
// of the residues, computed at compile time from the moduli.
#pragma once

#include <stdint.h>

#include "modular.h"

namespace mdg {

// Row of modulus i of the N-moduli system.
__host__ __device__ constexpr int mod_row(int N, int i) { return N * (N - 1) / 2 + i; }
constexpr int kModRows = kMaxModuli * (kMaxModuli + 1) / 2;

struct ModTables {
  double W[kModRows][kModLimbs] = {};           // W_i in 32-bit limbs, least significant first
  double M[kMaxModuli + 1][kModLimbs] = {};     // M likewise
  int chunks[kMaxModuli + 1] = {};              // four-limb chunks of M
  double r[kMaxModuli] = {};                    // 1 / m_i
  // residue constants of modulus i scaled by W_i^-1 (row mod_row(N, i)) and
  // unscaled (row kModRows + i): six dwords of bytes 256^j f mod m, then m and
  // 1 / m as floats
  uint32_t residue[kModRows + kMaxModuli][8] = {};
};

constexpr void mul_limbs(double (&x)[kModLimbs], int f) {
  uint64_t carry = 0;
  for (int j = 0; j < kModLimbs; ++j) {
    const uint64_t v = static_cast<uint64_t>(x[j]) * static_cast<uint64_t>(f) + carry;
    x[j] = static_cast<double>(v & 0xffffffffull);
    carry = v >> 32;
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

constexpr ModTables make_mod_tables() {
  ModTables t;
  t.M[0][0] = 1.0;
  for (int N = 1; N <= kMaxModuli; ++N) {
    const int mN = kModuli[N - 1];
    t.r[N - 1] = 1.0 / mN;
    residue_row(t.residue[kModRows + N - 1], 1, mN);
    for (int i = 0; i + 1 < N; ++i) {
      for (int j = 0; j < kModLimbs; ++j) t.W[mod_row(N, i)][j] = t.W[mod_row(N - 1, i)][j];
      mul_limbs(t.W[mod_row(N, i)], mN);
    }
    for (int j = 0; j < kModLimbs; ++j) t.W[mod_row(N, N - 1)][j] = t.M[N][j] = t.M[N - 1][j];
    mul_limbs(t.M[N], mN);
    for (int j = 0; j < kModLimbs; ++j)
      if (t.M[N][j] != 0.0) t.chunks[N] = j / 4 + 1;
    for (int i = 0; i < N; ++i) {
      int prod = 1;  // W_i mod m_i
      for (int j = 0; j < N; ++j)
        if (j != i) prod = prod * (kModuli[j] % kModuli[i]) % kModuli[i];
      residue_row(t.residue[mod_row(N, i)], inverse_mod(prod, kModuli[i]), kModuli[i]);
    }
  }
  return t;
}

// One copy per translation unit that uses it, in the device's constant memory.
static __constant__ const ModTables kModTables = make_mod_tables();

}  // namespace mdg
