// Level products on the int8 matrix cores by blocks of digit pairs.
//
// The product of an element pair is Z = sum over the kept digit pairs (p, q) of
// DA_p DB_q 2^(-w (p + q)), summed over k: a sum of integers, so any exact way
// of forming it gives the same limbs.  The kept pairs are covered by disjoint
// rectangles [p0, p0 + u) x [q0, q0 + v).  The digits of a rectangle are one
// signed integer per element, a = sum of DA_p 2^(w (p1 - p)) of w u bits, b of
// w v bits, and the rectangle contributes V 2^(-w (p1 + q1)) with V = sum_k a b.
//  - Residue groups: V is formed modulo N pairwise coprime moduli of at most 8
//    bits, one int8 product each (operands the balanced residues of a and b), and
//    recovered by the Chinese remainder theorem: V = sum_i y_i W_i - q M with
//    W_i = M / m_i and y_i = V W_i^-1 mod m_i (the factor W_i^-1 is folded into
//    A's residues, so the product's residue is y_i itself).  N grows with the
//    bits of V, w (u + v) + log2 k, while the pairs covered grow with u v: eight
//    by eight 13-bit digits take 29 products instead of 192.
//  - Direct groups: single pairs of one level, by sub-digits of 7 bits
//    (balanced, base 128) and Karatsuba's identity on them: c = ceil((w + 1) / 7)
//    sub-digits take c (c + 1) / 2 products (3 for 13-bit digits, against 6 or 7
//    residues), each summed in int32 over the level's pairs.
// Rectangles (or pairs) with the same p1 + q1 and bits share a group: their
// products are summed over a longer k range.
#pragma once

#include <stdint.h>

#include <memory>
#include <vector>

namespace mdg {

constexpr int kMaxModuli = 40;  // 291 bits; the next ones hold less than 6.2 bits
constexpr int kModLimbs = 10;   // 32-bit limbs of the product of all moduli
constexpr int kModMaxBlocks = 136;
constexpr int kModMaxPanels = 512;
constexpr int kModMaxGroups = 136;
constexpr int kModMaxJobs = 320;
constexpr int kModMaxDirect = kModMaxJobs;  // planes of the direct groups: one per direct job
constexpr int kModMaxChannelBlocks = 96;    // the residue groups' planes by sixteens, each group's apart
constexpr int kDirectTypes = 10;  // sub-digit products of a digit pair (4 sub-digits)
constexpr int kModMaxBits = 192;  // integer of a residue block
constexpr int kModTile = 256;     // output tile edge of the int8 products
constexpr int kModStage = 128;    // bytes of k per LDS stage

// The largest pairwise coprime integers up to 256, greedily from 256 down.
constexpr int kModuli[kMaxModuli] = {256, 255, 253, 251, 247, 241, 239, 233, 229, 227, 223, 217, 211, 199,
                                     197, 193, 191, 181, 179, 173, 167, 163, 157, 151, 149, 139, 137, 131,
                                     127, 113, 109, 107, 103, 101, 97,  89,  83,  79,  73,  71};

// Digits p0 .. p0 + u - 1 of an operand as one integer: bits lo .. lo + bits - 1
// of D; `count` int8 panels are made from it: residues modulo the first `count`
// moduli (residue, with the factors of the `count`-moduli system folded in when
// scaled), or the sub-digit types of one digit (direct), or sub-digit pick - 1 of
// one digit alone (scaled marks the top one).
struct ModBlock {
  uint16_t lo;
  uint8_t bits, count, residue, scaled, pick;
};

// One int8 product: panels a + i da of A times b + i db of B, i < nseg, summed;
// residue jobs (mod < kMaxModuli) store y as one byte, direct ones int32; out in
// units of one dword per four rows.
struct ModJob {
  uint16_t a, b;
  int16_t da, db;
  uint16_t nseg, mod, out;
};
constexpr int kDirectJob = 255;

// Output planes out .. of a group and the weight 2^shift of its value V in the
// accumulated integer N = sum_t G_t 2^(w (T - t)).
struct ModGroup {
  uint16_t shift, out;
  uint8_t residue, count;
};

struct ModPlan {
  std::vector<ModBlock> a, b;
  std::vector<ModJob> jobs;
  std::vector<ModGroup> groups;
  int pa = 0, pb = 0;    // panels of A and of B
  int planes = 0;        // dwords per four rows of all output planes
  int direct_bits = 0;   // w
  int64_t products = 0;  // int8 products of length k
  int directs = 0;       // planes of the direct groups
  int channels = 0;      // sixteens of planes of the residue groups
  double seconds = 0.0;  // of products, panels and planes at their rates, for choosing the path
};

// Levels in place: where the level planes G_t themselves are wanted (a caller
// workspace that may be read), each level is formed by one job over sub-digits of 7
// bits: with c of them, pass s = 0 .. 2c - 2 sums the products of sub-digits i + j = s
// of the level's pairs in int32 and adds 2^(7 s) times that to the level.  Panels:
// sub-digit i of digit p of A at i S + p, sub-digit j of digit q of B at j S + S - 1 - q,
// so that a level's pairs are one contiguous run for each (i, j).
struct LevelPlan {
  std::vector<ModBlock> a, b;
  int S = 0, T = 0, c = 0;
};
LevelPlan level_plan(int S, int T, int w);
constexpr int64_t kLevelsMaxN = int64_t{1} << 20;  // a tile's rows of a plane in 32-bit offsets
// 7-bit sub-digits of a w-bit digit (balanced, the last one up to 64 in magnitude).
inline int sub_digits(int w) { return w <= 7 ? 1 : (w + 7) / 7; }
// Whether the int32 sums of a pass hold for levels of up to `pairs` pairs: up to c runs of
// k products per pair.  A digit of at most 7 bits is its own sub-digit, up to 2^w - 1 in
// magnitude (products below 2^14); wider ones give balanced sub-digits of at most 64.
inline bool level_passes_exact(int pairs, int64_t k, int w) {
  const int64_t d = w <= 7 ? (int64_t{1} << w) - 1 : 64;
  return static_cast<double>(pairs) * sub_digits(w) * static_cast<double>(k) * static_cast<double>(d * d) <
         2147483648.0;
}

// The plan for the digit pairs p + q <= T of S digits of w bits and an m x k by
// k x n product; nullptr when none fits the limits above (or the int32 sums).  A plan
// that is returned is one that the accumulation takes (modular_accum_fits): the choice
// of the path asks nothing else about the planes after it has enqueued work.
std::shared_ptr<const ModPlan> modular_plan(int64_t m, int64_t n, int64_t k, int S, int T, int w);

// Whether the accumulation's tables hold the plan's planes (modular_accum.hip; host only).
bool modular_accum_fits(const ModPlan& pl, int w);
// Whether one launch of the split holds an m x k by k x n product (modular_split.hip; host only).
bool modular_split_fits(int64_t m, int64_t n, int64_t k);

constexpr int kModMaxWords = 15;  // 64-bit words of the accumulated integer

// The split's tiles: 16 lines by 128 values of k where the integer of an element is short,
// else 64; the panels of a tile are shared over up to eight blocks.
constexpr int kModSplitLines = 16;
inline bool mod_split_short(int L, int bits) { return (L <= 2 && bits <= 128) || (L <= 4 && bits <= 256); }
inline int64_t mod_split_tiles(int64_t m, int64_t n) {
  return (m + kModSplitLines - 1) / kModSplitLines + (n + kModSplitLines - 1) / kModSplitLines;
}
inline int64_t mod_split_shares(int64_t tiles) { return tiles >= 512 ? 1 : tiles > 64 ? 512 / tiles : 8; }

inline int64_t mod_kp(int64_t k) { return (k + kModStage - 1) / kModStage * kModStage; }
inline int64_t mod_rows(int64_t x) { return (x + kModTile - 1) / kModTile * kModTile; }
inline int64_t mod_quads(int64_t m) { return (m + 3) / 4; }

}  // namespace mdg
