// Context set-up: the jump-ahead tables of MRG32K3A, LFSR113 and the GM/GQ
// ensembles, computed once on the host when a context is created and then
// uploaded (the MT19937 polynomials are built in mt_poly.cpp).  A distance is
// applied as one matrix M^(d 2^(8 j)) per nonzero byte d, LFSR113 and GM/GQ
// distances above 64 bits as one ladder entry M^(2^b) per set bit b (the
// paper's jump-ahead sections decompose the distance in binary).
#include <cstring>
#include <vector>

#include "prand_impl.h"

namespace prand {
namespace {

typedef unsigned __int128 u128;

// ---------------------------------------------------------------- MRG32K3A
void mat3_sqr(const uint64_t* a, uint64_t* r, uint64_t m) {
  uint64_t t[9];
  for (int i = 0; i < 3; i++)
    for (int j = 0; j < 3; j++) {
      u128 acc = 0;
      for (int k = 0; k < 3; k++) acc += (u128)a[3 * i + k] * a[3 * k + j];
      t[3 * i + j] = (uint64_t)(acc % m);
    }
  std::memcpy(r, t, sizeof t);
}

void mat3_mul(const uint64_t* a, const uint64_t* b, uint64_t* r, uint64_t m) {
  uint64_t t[9];
  for (int i = 0; i < 3; i++)
    for (int j = 0; j < 3; j++) {
      u128 acc = 0;
      for (int k = 0; k < 3; k++) acc += (u128)a[3 * i + k] * b[3 * k + j];
      t[3 * i + j] = (uint64_t)(acc % m);
    }
  std::memcpy(r, t, sizeof t);
}
// a^e mod m for a 3x3 matrix
void mat3_pow(const uint64_t* a, uint64_t e, uint64_t* r, uint64_t m) {
  uint64_t p[9], acc[9] = {1, 0, 0, 0, 1, 0, 0, 0, 1};
  std::memcpy(p, a, sizeof p);
  for (; e; e >>= 1) {
    if (e & 1) mat3_mul(acc, p, acc, m);
    mat3_sqr(p, p, m);
  }
  std::memcpy(r, acc, sizeof acc);
}
}  // namespace

namespace {
// r = a b mod m (entries below m = 2^32 - c, c < 2^15), in 64-bit folds
void mat3_mul_fold(const uint32_t* a, const uint32_t* b, uint32_t* r, uint32_t c) {
  const uint64_t m = (1ull << 32) - c;
  uint32_t t[9];
  for (int i = 0; i < 3; i++)
    for (int j = 0; j < 3; j++) {
      uint64_t acc = 0;
      for (int k = 0; k < 3; k++) {
        const uint64_t v = (uint64_t)a[3 * i + k] * b[3 * k + j];
        acc += (v >> 32) * c + (uint32_t)v;
      }
      acc = (acc >> 32) * c + (uint32_t)acc;
      acc = (acc >> 32) * c + (uint32_t)acc;
      t[3 * i + j] = (uint32_t)(acc >= m ? acc - m : acc);
    }
  std::memcpy(r, t, sizeof t);
}
}  // namespace

// out [64][256][18]: A^(d 2^(8 j)) mod m1, then B^(d 2^(8 j)) mod m2
void build_mrg_bytes(uint32_t* out) {
  const uint32_t gen[2][9] = {{0, kMrgA12, kMrgM1 - kMrgA13n, 1, 0, 0, 0, 1, 0},
                              {kMrgA21, 0, kMrgM2 - kMrgA23n, 1, 0, 0, 0, 1, 0}};
  for (int h = 0; h < 2; h++) {
    const uint32_t c = h ? 0u - kMrgM2 : 0u - kMrgM1;
    uint32_t b[9], t[9];
    std::memcpy(b, gen[h], sizeof b);
    for (int j = 0; j < 64; j++) {
      for (int i = 0; i < 9; i++) t[i] = i % 4 == 0;
      for (int d = 0; d < 256; d++) {
        std::memcpy(out + ((size_t)j * 256 + d) * 18 + 9 * h, t, sizeof t);
        mat3_mul_fold(b, t, t, c);
      }
      std::memcpy(b, t, sizeof b);   // t = b^256
    }
  }
}

void build_mrg_section_table(uint64_t seclen, uint32_t* out) {
  const uint64_t A[9] = {0, kMrgA12, kMrgM1 - kMrgA13n, 1, 0, 0, 0, 1, 0};
  const uint64_t B[9] = {kMrgA21, 0, kMrgM2 - kMrgA23n, 1, 0, 0, 0, 1, 0};
  uint64_t SA[9], SB[9], MA[9], MB[9];
  mat3_pow(A, seclen, SA, kMrgM1);
  mat3_pow(B, seclen, SB, kMrgM2);
  std::memcpy(MA, SA, sizeof MA);
  std::memcpy(MB, SB, sizeof MB);
  for (int j = 1; j < kSectionTableRows + 1; j++) {
    for (int i = 0; i < 9; i++) {
      out[(j - 1) * 18 + i] = (uint32_t)MA[i];
      out[(j - 1) * 18 + 9 + i] = (uint32_t)MB[i];
    }
    mat3_mul(SA, MA, MA, kMrgM1);
    mat3_mul(SB, MB, MB, kMrgM2);
  }
}

// ----------------------------------------------------------------- LFSR113
namespace {
constexpr int kLfP[4] = {31, 29, 28, 25};
constexpr int kLfQ[4] = {6, 2, 13, 3};
constexpr int kLfS[4] = {18, 2, 7, 13};

uint32_t lfsr_word_step(uint32_t z, int c) {
  const uint32_t mask = 0xFFFFFFFFu << (32 - kLfP[c]);
  return ((z & mask) << kLfS[c]) ^ (((z << kLfQ[c]) ^ z) >> (kLfP[c] - kLfS[c]));
}
uint32_t f2_apply(const uint32_t* cols, uint32_t v) {
  uint32_t r = 0;
  while (v) {
    int j = __builtin_ctz(v);
    r ^= cols[j];
    v &= v - 1;
  }
  return r;
}
}  // namespace

namespace {
// a matrix by the bytes of the word it is applied to
struct F2Bytes {
  uint32_t t[4][256];
  explicit F2Bytes(const uint32_t* cols) {
    for (int q = 0; q < 4; q++) {
      t[q][0] = 0;
      for (int x = 1; x < 256; x++) t[q][x] = t[q][x & (x - 1)] ^ cols[8 * q + __builtin_ctz(x)];
    }
  }
  uint32_t apply(uint32_t v) const { return t[0][v & 255] ^ t[1][v >> 8 & 255] ^ t[2][v >> 16 & 255] ^ t[3][v >> 24]; }
};

// columns of T_c^(d 2^(e + 8 j)) for every byte position j < 8 and value d
// (row [j][d], 128 words, the layout of the section tables)
void lfsr_bytes(int e, uint32_t* out) {
  for (int c = 0; c < 4; c++) {
    uint32_t b[32], t[32], m[32];
    for (int j = 0; j < 32; j++) b[j] = lfsr_word_step(1u << j, c);
    for (int i = 0; i < e; i++) {   // b = T_c^(2^e)
      for (int j = 0; j < 32; j++) t[j] = f2_apply(b, b[j]);
      std::memcpy(b, t, sizeof t);
    }
    for (int pos = 0; pos < 8; pos++) {
      const F2Bytes by(b);
      for (int j = 0; j < 32; j++) m[j] = 1u << j;   // d = 0: identity
      for (int d = 0; d < 256; d++) {
        std::memcpy(out + (((size_t)pos * 256 + d) * 4 + c) * 32, m, sizeof m);
        for (int j = 0; j < 32; j++) m[j] = by.apply(m[j]);
      }
      std::memcpy(b, m, sizeof b);   // m = b^256
    }
  }
}
}  // namespace

void build_lfsr_jumps(uint32_t* out) {
  for (int c = 0; c < 4; c++) {
    uint32_t cols[32];
    for (int j = 0; j < 32; j++) cols[j] = lfsr_word_step(1u << j, c);
    for (int b = 0; b < kLadder; b++) {
      std::memcpy(out + ((size_t)b * 4 + c) * 32, cols, sizeof cols);
      uint32_t sq[32];
      for (int j = 0; j < 32; j++) sq[j] = f2_apply(cols, cols[j]);
      std::memcpy(cols, sq, sizeof sq);
    }
  }
  lfsr_bytes(0, out + (size_t)kLadder * 128);
}

void build_lfsr_byte_table(uint32_t* out) { lfsr_bytes(kLfsrByteE, out); }

void build_lfsr_section_table(uint64_t seclen, uint32_t* out) {
  for (int c = 0; c < 4; c++) {
    // S = T_c^seclen by squaring; columns of the composition P o Q are P
    // applied to the columns of Q
    uint32_t p[32], s[32], m[32], t[32];
    for (int j = 0; j < 32; j++) {
      p[j] = lfsr_word_step(1u << j, c);
      s[j] = 1u << j;
    }
    for (uint64_t e = seclen; e; e >>= 1) {
      if (e & 1) {
        for (int j = 0; j < 32; j++) t[j] = f2_apply(p, s[j]);
        std::memcpy(s, t, sizeof t);
      }
      for (int j = 0; j < 32; j++) t[j] = f2_apply(p, p[j]);
      std::memcpy(p, t, sizeof t);
    }
    std::memcpy(m, s, sizeof m);
    for (int j = 1; j < kSectionTableRows + 1; j++) {
      std::memcpy(out + ((size_t)(j - 1) * 4 + c) * 32, m, sizeof m);
      for (int i = 0; i < 32; i++) t[i] = f2_apply(s, m[i]);
      std::memcpy(m, t, sizeof t);
    }
  }
}

// ------------------------------------------------------------------- GM/GQ
namespace {
struct Mat2 {
  uint64_t a, b, c, d;
};
Mat2 mat2_mul(const Mat2& x, const Mat2& y, uint64_t p) {
  return Mat2{(uint64_t)(((u128)x.a * y.a + (u128)x.b * y.c) % p), (uint64_t)(((u128)x.a * y.b + (u128)x.b * y.d) % p),
              (uint64_t)(((u128)x.c * y.a + (u128)x.d * y.c) % p), (uint64_t)(((u128)x.c * y.b + (u128)x.d * y.d) % p)};
}
uint64_t pow_mod(uint64_t x, uint64_t e, uint64_t p) {
  uint64_t r = 1 % p;
  for (; e; e >>= 1) {
    if (e & 1) r = (uint64_t)((u128)r * x % p);
    x = (uint64_t)((u128)x * x % p);
  }
  return r;
}
}  // namespace

// out [8][8][256][4]: M^(d 2^(kGmByteE[g] + 8 j)) mod p; neg [8][4]: M^(-n0)
// mod p (the inverse of M^n0 through the adjugate and det^(p-2), p prime),
// the identity where n0 = 0
void build_gm_byte_tables(uint64_t* out, uint64_t* neg) {
  for (int g = 0; g < 8; g++) {
    const GmParams& P = kGmParams[g];
    const uint64_t p = P.p;
    const Mat2 m{P.k % p, (p - P.q % p) % p, 1, 0};
    Mat2 b = m;
    for (int i = 0; i < kGmByteE[g]; i++) b = mat2_mul(b, b, p);
    for (int pos = 0; pos < 8; pos++) {
      Mat2 t{1, 0, 0, 1};
      for (int d = 0; d < 256; d++) {
        uint64_t* o = out + (((size_t)g * 8 + pos) * 256 + d) * 4;
        o[0] = t.a; o[1] = t.b; o[2] = t.c; o[3] = t.d;
        t = mat2_mul(t, b, p);
      }
      for (int i = 0; i < 8; i++) b = mat2_mul(b, b, p);
    }
    Mat2 f{1, 0, 0, 1};
    for (int i = 0; i < P.n0; i++) f = mat2_mul(f, m, p);
    const uint64_t det = (uint64_t)(((u128)f.a * f.d + (u128)(p - f.b) * f.c) % p);
    const uint64_t inv = pow_mod(det, p - 2, p);
    uint64_t* o = neg + (size_t)g * 4;
    o[0] = (uint64_t)((u128)f.d * inv % p);
    o[1] = (uint64_t)((u128)((p - f.b) % p) * inv % p);
    o[2] = (uint64_t)((u128)((p - f.c) % p) * inv % p);
    o[3] = (uint64_t)((u128)f.a * inv % p);
  }
}

void build_gm_jumps(uint64_t* out) {
  for (int g = 0; g < 8; g++) {
    const GmParams& P = kGmParams[g];
    const uint64_t p = P.p;
    uint64_t* const o = out + (size_t)g * kJumpRows * 4;
    auto put = [&](size_t row, const Mat2& m) {
      const uint64_t v[4] = {m.a, m.b, m.c, m.d};
      std::memcpy(o + 4 * row, v, sizeof v);
    };
    const Mat2 m{P.k % p, (p - P.q % p) % p, 1, 0};
    Mat2 b = m;
    for (int i = 0; i < kLadder; i++) {
      put(i, b);
      b = mat2_mul(b, b, p);
    }
    b = m;
    for (int pos = 0; pos < 8; pos++) {
      Mat2 t{1, 0, 0, 1};
      for (int d = 0; d < 256; d++) {
        put(kLadder + 256 * pos + d, t);
        t = mat2_mul(t, b, p);
      }
      b = t;
    }
  }
}

namespace {
// digits of v in [-2^(b-1), 2^(b-1)), least first; false when `n` do not hold it
bool balanced(__int128 v, int b, int n, int* d) {
  const int half = 1 << (b - 1);
  for (int m = 0; m < n; m++) {
    d[m] = (int)((v + half) & (2 * half - 1)) - half;
    v = (v - d[m]) >> b;
  }
  return v == 0;
}

// Digits of a coefficient a < p: of the representations a + t p that `n`
// digits hold, one whose positive digits have a small sum (they lower the
// result, see dev_gmx.h), then a small sum of magnitudes.
void gmx_digits(uint64_t a, uint64_t p, int b, int n, int* best) {
  int score = 1 << 30;
  int d[8];
  // `n` digits hold the values of magnitude below 2^(b n - 1) (1 + 2 / 2^b)
  const __int128 reach = ((__int128)1 << (b * n - 1)) + ((__int128)1 << (b * n - b));
  const int most = (int)(reach / p < 40 ? reach / p + 1 : 40);
  for (int t = -most; t <= most; t++) {
    if (!balanced((__int128)a + (__int128)t * p, b, n, d)) continue;
    int s = 0;
    for (int m = 0; m < n; m++) s += d[m] > 0 ? 3 * d[m] : -d[m];
    if (s < score) {
      score = s;
      std::memcpy(best, d, n * sizeof *d);
    }
  }
}

// v as f16: |v| < 65536, at most 11 significant bits
uint16_t gmx_half(int v) {
  if (!v) return 0;
  const uint32_t m = (uint32_t)(v < 0 ? -v : v);
  const int top = 31 - __builtin_clz(m);   // m in [2^top, 2^(top + 1))
  const uint32_t frac = top > 10 ? m >> (top - 10) : m << (10 - top);
  return (uint16_t)((v < 0 ? 0x8000u : 0u) | (uint32_t)(top + 15) << 10 | (frac & 0x3FFu));
}
}  // namespace

// Powers M^j and the coefficient operands of the matrix instructions: lane l
// holds column l % 32 (step 32 g + l % 32 + 1) of the digits of alpha (lanes
// 0..31, products 0..7) or beta (lanes 32..63, products 8..15).
void build_gmx_tables(GmxTable* out) {
  for (int g = 0; g < 8; g++) {
    const GmParams& P = kGmParams[g];
    const uint64_t p = P.p;
    const int n = kGmxShape[g].digits, b = kGmxShape[g].bits;
    GmxTable& T = out[g];
    std::memset(T.coef, 0, sizeof T.coef);
    const Mat2 m{P.k % p, (p - P.q % p) % p, 1, 0};
    Mat2 r{1, 0, 0, 1};
    for (int j = 0; j <= kGmxSteps; j++) {
      const uint64_t row[4] = {r.a, r.b, r.c, r.d};
      std::memcpy(T.mat + 4 * j, row, sizeof row);
      for (int h = 0; j && h < 2; h++) {
        int d[8] = {0};
        gmx_digits(h ? r.b : r.a, p, b, n, d);
        uint16_t* o = T.coef + ((size_t)(j - 1) / 32 * 64 + (j - 1) % 32 + 32 * h) * 8;
        for (int i = 0; i < 8; i++)
          if (gmx_below(b, i) < n)
            o[i] = gmx_half(d[n - 1 - gmx_below(b, i)] * gmx_factor(kGmxShape[g].width, i));
      }
      r = mat2_mul(m, r, p);
    }
  }
}

}  // namespace prand

// Not in the public header (a test hook): the table of one GM/GQ generator
// (index 0 GM19 .. 7 GQ58.4): the powers M^j, and the digits of step j =
// 1 .. kGmxSteps read back from the operands, digits[2 (j - 1) + h][m] (h = 0:
// of x^(n), 1: of x^(n-1); 8 digits, least first).  dims: steps, digits,
// positions, bits of a position, offset, bits of a digit, doubled top.  0 on
// success; -1 when a product without a digit has a coefficient, or a digit's two
// parts differ.
extern "C" int prand_internal_gmx_table(int g, uint64_t* mat, int16_t* digits, int* dims) {
  if (g < 0 || g >= 8 || !mat || !digits || !dims) return PRAND_EINVAL;
  std::vector<prand::GmxTable> t(8);
  prand::build_gmx_tables(t.data());
  const prand::GmxShape& S = prand::kGmxShape[g];
  std::memcpy(mat, t[g].mat, sizeof t[g].mat);
  dims[0] = prand::kGmxSteps;
  dims[1] = S.digits;
  dims[2] = S.positions;
  dims[3] = S.width;
  dims[4] = S.delta;
  dims[5] = S.bits;
  dims[6] = S.top;
  for (int j = 0; j < prand::kGmxSteps; j++)
    for (int h = 0; h < 2; h++) {
      int16_t* d = digits + (2 * j + h) * 8;
      std::memset(d, 0, 8 * sizeof *d);
      const uint16_t* o = t[g].coef + ((size_t)(j / 32) * 64 + j % 32 + 32 * h) * 8;
      for (int i = 0; i < 8; i++) {
        // the f16 value, an integer, over the factor
        const int exp = (o[i] >> 10 & 31) - 15, m = 1024 | (o[i] & 1023);
        const int v = o[i] ? (o[i] & 0x8000 ? -1 : 1) * (m << exp >> 10) : 0;
        const int below = prand::gmx_below(S.bits, i), factor = prand::gmx_factor(S.width, i);
        if (below >= S.digits ? v != 0 : v % factor != 0) return -1;
        if (below >= S.digits) continue;
        int16_t& at = d[S.digits - 1 - below];
        // the second part of a digit repeats the first
        if (S.width != 11 && (i & 1) && at != v / factor) return -1;
        at = (int16_t)(v / factor);
      }
    }
  return 0;
}
