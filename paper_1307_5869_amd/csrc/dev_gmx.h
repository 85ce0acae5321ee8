// GM/GQ generation by matrix instructions.
//
// Step n + j of an element is a fixed linear combination of its two state
// values, x^(n+j) = alpha_j x^(n) + beta_j x^(n-1) (mod p), and its digit
// floor(2^v x / p) is the top v bits of the fraction x^(n+j) / p.  With
// alpha_j = sum_m a_jm 2^(b m) (and beta_j likewise) in b-bit digits a_jm of
// both signs, the fraction is
//    sum_m a_jm frac(2^(b m) x^(n) / p) + the same of x^(n-1)   (mod 1),
// a product of a constant matrix of small integers (32 steps by digits) with
// data of the state (digits by elements): the work of
// v_mfma_f32_32x32x16_f16, up to 8 digits of both state values.
//
// The fractions are cut to TB bits and these into L positions of 11 bits.  The
// 11 bits of a position are the f16 operand as they stand (below 2048 an f16's
// bits are its value over 2^-24: a subnormal, or the first normal binade), the
// digits are held times 256, so that sums are whole multiples of 2^-16.  They
// are kept at 192 + s 2^-16, |s| < 2^22, where the f32's last bit is 2^-16:
// every sum is exact and the low bits of the register's word are s.  The sums
// chain: position i + 1 starts from floor(s_i / 2^11), one multiply-add that
// rounds toward zero (the mode is set around the loop), and the top sum holds
// the digit: in bits 8 - v .. 7 of its word, or, where the fractions need all
// bits of the top position, in the second byte, the top position's data and
// carry doubled (GM55: bits 8 .. 11).  GM19's four 5-bit digits leave room for
// positions of 14 bits, each as two parts of 7 (the digit times 2 and times 256,
// sums of 2^-23 around 1.5), and two positions are enough (bit 14).
//
// Exactness.  Cutting a fraction loses e in [0, 1] units of 2^-TB, so the
// result is the true fraction (2^TB units) plus kDelta, plus at most
// N = sum of |a| over the negative digits of the step, minus at most P, the
// sum of its positive ones.  The true 2^v x / p is never closer than
// 1 / p to the integer above it, so the digit is exact when P <= kDelta and
// kDelta + N < 2^TB / (2^v p): the tables' digits are chosen for that (among
// the representations alpha + t p), and a CPU test checks it for every step,
// as it checks that no sum leaves the 2^22.
//
// One wavefront holds 32 elements: one stream of a v = 1 ensemble, four of 8
// elements, two of GQ58.3 (24 rows used).  Lane e < 32 keeps x^(n) of row e,
// lane e + 32 its x^(n-1); the data of J = 256 steps are made at once and the
// state then moves J steps on (one 2 x 2 product mod p).  The results come
// with the step along the lanes, so words are stored 64 consecutive ones at a
// time, with no LDS.
//
// Bound: power, then issue.  Per 1024 element steps L matrix instructions of
// 32 cycles, 16 (L - 1) carries and about 20 operations to gather the digits;
// the matrix instructions overlap little with the carries of other wavefronts,
// and with random operands the clock falls to 1.8 GHz (2.3-2.4 GHz in the
// kernels this replaced).  The same by v_mfma_i32_32x32x32_i8, each 11 bits as
// two bytes, holds half the coefficient bits per instruction: GM55 and GM61
// then take two per position.  2^30 words (65536 streams, u32), before (one
// lane per element and a ballot per word, or one lane per section), by i8, and
// now: GM29 7.3, 5.3, 4.9 ms; GM31 7.3, 5.2, 5.0; GQ58.1 7.3, 5.25, 4.9; GM55 3.9, 3.1, 2.25;
// GQ58.3 4.2, 3.3, 3.2; GQ58.4 2.6, 1.6, 1.55; GM19 4.1, 4.2, 3.3; GM61 10.5, 12.4, 8.9.
#pragma once

#include "dev_gm.h"

namespace prand {
namespace gm {

typedef int I4 __attribute__((ext_vector_type(4)));
typedef float F16 __attribute__((ext_vector_type(16)));
typedef _Float16 H2 __attribute__((ext_vector_type(2)));
typedef _Float16 H8 __attribute__((ext_vector_type(8)));

template <int G>
struct Mx {
  static constexpr int S = kGmParams[G].s, V = kGmParams[G].v, T = kGmParams[G].t;
  static constexpr int E = kGmxShape[G].e;            // p = 2^E - C
  static constexpr uint64_t C = kGmxShape[G].c, P = kGmParams[G].p;
  static constexpr int B = kGmxShape[G].bits, D = kGmxShape[G].digits, L = kGmxShape[G].positions;
  static constexpr bool TOP = kGmxShape[G].top != 0;
  static constexpr int W = kGmxShape[G].width;
  static constexpr int TB = W * (L - 1) + (TOP ? W : 8);   // bits of a fraction
  static constexpr int WF = TB + B * (D - 1);         // bits of x / p that the digits reach
  static constexpr int NW = (WF + 31) / 32;           // 32-bit words of it
  static constexpr int NA = B == 8 && D <= 4 ? 2 : 4;   // data words per position (the others are zero)
  static constexpr int Q = S == 32 ? 1 : (S == 8 ? 4 : 2);   // streams per wavefront
  static constexpr int kDelta = kGmxShape[G].delta;
  // a sum s is held as kZero + s kUnit, kUnit the last bit of kZero
  static constexpr float kUnit = gmx_factor(W, 0) * 0x1p-24f, kZero = 0x1.8p23f * kUnit;
};

// row of the 32-element tile -> stream of the wavefront and element (-1: idle
// row).  The result of row 8 t + 4 h + b is in accumulator register 4 t + b of
// half h of the wavefront; the bit orders below follow from how words()
// gathers the registers.
template <int G>
__device__ __forceinline__ int gmx_row_stream(int row) {
  return Mx<G>::Q == 1 ? 0 : (Mx<G>::Q == 4 ? row >> 3 : row >> 4);
}
template <int G>
__device__ __forceinline__ int gmx_row_element(int row) {
  const int t = row >> 3, h = (row >> 2) & 1, b = row & 3;
  if constexpr (Mx<G>::S == 32) return 31 - (8 * b + 4 * (1 - h) + 3 - t);
  else if constexpr (Mx<G>::S == 8) return 2 * (3 - b) + h;
  else return (t & 1) ? (h ? -1 : 8 + 3 - b) : 4 * h + 3 - b;
}

// m0 a + m1 b mod p, all below p
template <int G>
__device__ __forceinline__ uint64_t gmx_mulsum(uint64_t m0, uint64_t a, uint64_t m1, uint64_t b) {
  using M = Mx<G>;
  if constexpr (M::E > 32) {
    return fold_special<G>((u128)m0 * a + (u128)m1 * b, M::E, M::C, M::P);
  } else {
    constexpr uint64_t mask = (1ull << M::E) - 1;
    const uint64_t t = (uint64_t)(uint32_t)m0 * (uint32_t)a + (uint64_t)(uint32_t)m1 * (uint32_t)b;   // < 2^63
    const uint64_t u = (t & mask) + M::C * (t >> M::E);
    const uint32_t w = (uint32_t)(u & mask) + (uint32_t)M::C * (uint32_t)(u >> M::E);   // < p + 32
    return w >= (uint32_t)M::P ? w - (uint32_t)M::P : w;
  }
}

// floor(2^WF x / p) or one less, as 32-bit words: x / p = x 2^-E (1 + C 2^-E
// + C^2 2^-2E + ...); with C = 1 the terms are x's bits repeated
template <int G>
__device__ __forceinline__ void gmx_fraction(uint64_t x, uint32_t (&f)[Mx<G>::NW]) {
  using M = Mx<G>;
#pragma unroll
  for (int i = 0; i < M::NW; i++) f[i] = 0;
  if constexpr (G == 4) {
    static_assert(G != 4 || M::WF == 130, "GM61 fraction");
    const u128 lo = ((u128)x << 69) | ((u128)x << 8) | (x >> 53);
    f[0] = (uint32_t)lo;
    f[1] = (uint32_t)(lo >> 32);
    f[2] = (uint32_t)(lo >> 64);
    f[3] = (uint32_t)(lo >> 96);
    f[4] = (uint32_t)(x >> 59);
  } else if constexpr (G == 3) {
    static_assert(G != 3 || M::WF == 114, "GM55 fraction");
    const u128 lo = ((u128)x << 63) + ((u128)(129ull * x) << 12) + (uint64_t)(((u128)x * 16641u) >> 39);
    f[0] = (uint32_t)lo;
    f[1] = (uint32_t)(lo >> 32);
    f[2] = (uint32_t)(lo >> 64);
    f[3] = (uint32_t)(lo >> 96);
  } else if constexpr (G == 0) {
    static_assert(G != 0 || M::WF == 43, "GM19 fraction");
    const uint64_t lo = (x << 24) | (x << 5) | (x >> 14);
    f[0] = (uint32_t)lo;
    f[1] = (uint32_t)(lo >> 32);
  } else if constexpr (G == 2) {
    static_assert(G != 2 || M::WF == 69, "GM31 fraction");
    const uint32_t v = (uint32_t)x;
    f[0] = (v << 7) | (v >> 24);
    f[1] = (v << 6) | (v >> 25);
    f[2] = v >> 26;
  } else {   // p = 2^29 - 3
    constexpr int sh = M::WF - 29;
    static_assert(!(G == 1 || G >= 5) || (sh >= 35 && sh <= 40), "2^29 - 3 fraction");
    const uint64_t lo = (x << sh) + ((3 * x) << (sh - 29)) + ((9 * x) >> (58 - sh));
    f[0] = (uint32_t)lo;
    f[1] = (uint32_t)(lo >> 32);
    f[2] = (uint32_t)(x >> (64 - sh));
    // (x << sh) drops the bits above 64 into f[2]; the two smaller terms
    // may carry into it
    f[2] += (lo < (x << sh)) ? 1u : 0u;
  }
}

// 32 bits of f from bit `at`
template <int N>
__device__ __forceinline__ uint32_t gmx_bits(const uint32_t (&f)[N], int at) {
  const int w = at >> 5, b = at & 31;
  const uint32_t lo = w < N ? f[w] : 0, hi = w + 1 < N ? f[w + 1] : 0;
  return b ? __builtin_amdgcn_alignbit(hi, lo, b) : lo;
}

// the data operands of a state value: position s; word w holds the 11 bits
// from 11 s + b gmx_below(2 w), and those 16 bits above; or the 7 bits from
// 14 s + b gmx_below(2 w) and the 7 above
template <int G>
__device__ __forceinline__ void gmx_operands(uint64_t x, I4 (&A)[Mx<G>::L]) {
  using M = Mx<G>;
  uint32_t f[M::NW];
  gmx_fraction<G>(x, f);
#pragma unroll
  for (int s = 0; s < M::L; s++) {
#pragma unroll
    for (int w = 0; w < 4; w++) {
      uint32_t v = 0;
      if (w < M::NA) v = gmx_bits(f, M::W * s + M::B * gmx_below(M::B, 2 * w));
      v = M::W == 11 ? v & 0x07FF07FFu : (v & 0x7Fu) | ((v << 9) & 0x7F0000u);
      if (M::TOP && s == M::L - 1) {
        const H2 h = __builtin_bit_cast(H2, v);
        v = __builtin_bit_cast(uint32_t, (H2)(h + h));
      }
      A[s][w] = (int)v;
    }
  }
}

// top sums of 32 steps (coefficients B) for the wavefront's rows; c: the
// offset in every element; rounding toward zero
template <int G>
__device__ __forceinline__ F16 gmx_chain(const I4 (&A)[Mx<G>::L], const I4& B, F16 c) {
  using M = Mx<G>;
#pragma unroll
  for (int s = 0; s < M::L; s++) {
    if (s) {
      const float scale = 1.0f / (1 << (M::W - (M::TOP && s == M::L - 1 ? 1 : 0)));
#pragma unroll
      for (int i = 0; i < 16; i++) c[i] = __builtin_fmaf(c[i], scale, M::kZero - M::kZero * scale);
    }
    c = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(H8, A[s]), __builtin_bit_cast(H8, B), c, 0, 0, 0);
  }
  return c;
}

// the digits' bytes of registers 4 t .. 4 t + 3 as the four bytes of a word
// (byte 0, the digit on top; or byte 1, GM55's digit in its lower half, GM19's
// in bit 6)
template <int G>
__device__ __forceinline__ uint32_t gmx_bytes(const F16& c, int t) {
  constexpr uint32_t byte = Mx<G>::TOP ? 1 : 0;
  auto word = [&](int i) { return __float_as_uint(c[4 * t + i]); };
  uint32_t r = __builtin_amdgcn_perm(word(1), word(0), 0x0c0c0400u + 0x0101u * byte);
  r = __builtin_amdgcn_perm(word(2), r, 0x0c040100u + 0x010000u * byte);
  return __builtin_amdgcn_perm(word(3), r, 0x04020100u + 0x01000000u * byte);
}
__device__ __forceinline__ uint32_t gmx_select(uint32_t a, uint32_t b, uint32_t mask) {
  return __builtin_amdgcn_bitop3_b32(a, b, mask, 0xE4);   // (a & mask) | (b & ~mask)
}

struct Swapped {
  uint32_t a, b;   // lower half: a's and b's lower-half value of the first; upper half: of the second
};
// halves exchanged: .a = first's lower half, then second's lower half; .b =
// first's upper half, then second's upper half
__device__ __forceinline__ Swapped gmx_swap(uint32_t first, uint32_t second) {
  const auto r = __builtin_amdgcn_permlane32_swap(first, second, false, false);
  return Swapped{r[0], r[1]};
}
// both halves' 64-bit values in every lane
__device__ __forceinline__ void gmx_both(uint64_t x, uint64_t& lower, uint64_t& upper) {
  const Swapped lo = gmx_swap((uint32_t)x, (uint32_t)x), hi = gmx_swap((uint32_t)(x >> 32), (uint32_t)(x >> 32));
  lower = ((uint64_t)hi.a << 32) | lo.a;
  upper = ((uint64_t)hi.b << 32) | lo.b;
}

// f32 rounding toward zero, or to nearest again (bits 1:0 of the mode
// register).  What else rounds in f32 in between, the conversions of outputs, is
// exact in either mode; no integer is divided there (the compiler's division is
// by f32 reciprocals), so sec() of gmx_wave must be made beforehand.
template <bool kZero>
__device__ __forceinline__ void gmx_round() {
  constexpr int kModeBits1to0 = 1 | 0 << 6 | (2 - 1) << 11;
  __builtin_amdgcn_s_setreg(kModeBits1to0, kZero ? 3 : 0);
}

// a value that is the same in every lane, in scalar registers
__device__ __forceinline__ uint64_t gmx_uniform(uint64_t v) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return ((uint64_t)hi << 32) | lo;
}

// one stream or section of a wavefront (uniform across it): n outputs from
// *in moved `start` outputs on; n = 0: none
struct GmxSec {
  const GmState* in;
  uint64_t start, n;
  char* out;
  GmState* sout;   // the state after n outputs (null: not wanted)
};

// LDS words per wavefront (the exact first steps of composite moduli)
constexpr int kGmxLds = 64;

// 12 bits of four bytes' top three bits, byte 3 first
__device__ __forceinline__ uint32_t gmx_pack3(uint32_t p) {
  const uint32_t z = p >> 5;
  const uint32_t y = (z & 0x00070007u) | ((z >> 5) & 0x00380038u);
  return (y & 0x3Fu) | (y >> 10);
}

// output word i in the element type DT, or in `dtype` where DT is kAnyType (a
// kernel for tasks of every generator and type: one copy of each generator's
// code)
constexpr int kAnyType = -1;
template <int DT>
__device__ __forceinline__ void gmx_put(void* out, uint64_t i, uint32_t w, int dtype) {
  if constexpr (DT != kAnyType) {
    put<DT>(out, i, w);
  } else {
    if (dtype == PRAND_F64) {
      put<PRAND_F64>(out, i, w);
    } else {
      const uint32_t f = __float_as_uint((float)(w >> 8) * 0x1p-24f);
      put<PRAND_U32>(out, i, dtype == PRAND_F32 ? f : w);
    }
  }
}

// Generate the wavefront's streams; sec(q) gives stream q < Mx<G>::Q.  A
// stream's input state is read before its output state is written, so they
// may be the same object.  kJump = false: every start is 0.  lds: kGmxLds
// words of this wavefront.  sec() is called in the loop too, under its rounding
// mode: it divides nothing.  dtype (uniform): read where DT is kAnyType.  All 64
// lanes must call.
template <int G, int DT, bool kJump, class SecOf>
__device__ __forceinline__ void gmx_wave(SecOf&& sec, const GmxTable* __restrict__ table,
                                         const uint64_t* __restrict__ ladder, uint32_t* lds, int dtype = DT) {
  using M = Mx<G>;
  using E = Eng<G>;
  constexpr int J = kGmxSteps;
  const int lane = threadIdx.x & 63;
  const bool upper = lane >= 32;
  const int q = gmx_row_stream<G>(lane & 31), e = gmx_row_element<G>(lane & 31);
  GmxSec mine = sec(0);
#pragma unroll
  for (int k = 1; k < M::Q; k++)
    if (q == k) mine = sec(k);
  const bool live = e >= 0 && mine.n != 0;

  // start values of this row, in both halves
  uint64_t xc = 0, xp = 0;
  uint32_t off0 = 0;   // GQ58.3: words of the first 8-step block already used
  if (live) off0 = load_at<G, kJump>(mine.in, e, mine.start, xc, xp, ladder);
  // outputs are counted from the block boundary where the state sits: frame
  // outputs off0 .. total - 1 are wanted
  const uint64_t total = live ? off0 + mine.n : 0;
  const uint64_t save_at = (G == 6) ? 8 * (total / 9) : total;   // steps to the output state
  const uint32_t off_end = (G == 6) ? (uint32_t)(total % 9) : 0u;
  uint64_t need = (G == 6) ? 8 * ((total + 8) / 9) : total;      // steps to run
  if constexpr (M::Q > 1) {
    for (int o = 4; o < 32; o <<= 1) {
      const uint64_t other = __shfl_xor(need, o);
      need = other > need ? other : need;
    }
  }
  need = ((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(need >> 32)) << 32) |
         (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)need);
  GmState* const sout = live ? mine.sout : nullptr;
  bool saved = false;
  // the output state of this row (the lower half writes x^(n), the upper
  // x^(n-1)); rows of element 0 clear the unused slots and set the offset
  auto save = [&](uint64_t v) {
    (upper ? sout->xp : sout->xc)[e] = v;
    if (M::S < 32 && e == 0)
      for (int i = M::S; i < 32; i++) (upper ? sout->xp : sout->xc)[i] = 0;
    if (e == 0 && !upper) {
      sout->off = off_end;
      sout->pad = 0;
    }
    saved = true;
  };
  if (G == 6 && sout && save_at == 0) save(upper ? xp : xc);

  // off0 and total of stream k, in every lane
  auto frame_of = [&](int k, uint64_t& o0, uint64_t& tot) {
    const GmxSec s = sec(k);
    o0 = (G == 6) ? (uint32_t)__builtin_amdgcn_readlane(off0, 16 * k) : 0;
    tot = s.n ? o0 + s.n : 0;
  };

  // composite moduli: n0 exact steps unless every element has collapsed
  uint64_t t = 0;
  if constexpr (E::kComposite) {
    constexpr int K = kGmParams[G].n0;
    constexpr int KW = K * M::S * M::V / 32;   // words they make
    static_assert(KW * M::Q <= kGmxLds && K * M::S * M::V % 32 == 0, "exact steps make whole words");
    if (!__all(!live || (E::collapsed(xc) && E::collapsed(xp)))) {
      if (lane < KW * M::Q) lds[lane] = 0;
      wave_lds_sync();
#pragma unroll 1
      for (int u = 0; u < K; u++) {
        const uint64_t nx = E::slow_step(xc, xp);
        xp = xc;
        xc = nx;
        if (live && !upper) {
          const uint32_t d = E::slow_digit(nx);
          const int bit = u * M::S * M::V + M::V * e;   // stream bit of the digit's top bit
          uint32_t* w = lds + q * KW + (bit >> 5);
          const int r = 32 - M::V - (bit & 31);
          if (r >= 0) {
            atomicOr(w, d << r);
          } else {
            atomicOr(w, d >> -r);
            atomicOr(w + 1, d << (32 + r));
          }
        }
        if (sout && (uint64_t)(u + 1) == save_at) save(upper ? xp : xc);
      }
      wave_lds_sync();
#pragma unroll
      for (int k = 0; k < M::Q; k++) {
        uint64_t o0, tot;
        frame_of(k, o0, tot);
        if (lane < KW && (uint64_t)lane >= o0 && (uint64_t)lane < tot)
          gmx_put<DT>(sec(k).out, lane - o0, lds[k * KW + lane], dtype);
      }
      wave_lds_sync();
      t = K;
    }
  }
  // from here each lane keeps one value of its row, below p
  uint64_t x = (upper ? xp : xc) >> M::T;
  x = x >= M::P ? x - M::P : x;

  const uint64_t* const mats = table->mat;
  const I4* const coef = (const I4*)table->coef + lane;
  uint64_t mj0 = mats[4 * J + (upper ? 2 : 0)], mj1 = mats[4 * J + (upper ? 3 : 1)];
  F16 offset;
#pragma unroll
  for (int i = 0; i < 16; i++) offset[i] = M::kZero + M::kDelta * M::kUnit;
  // v = 1: kept in registers of its own, not made again for every chain (1-3 %)
  if constexpr (M::S == 32) asm volatile("" : "+v"(offset));
  gmx_round<true>();
  for (; t < need; t += J) {
    I4 A[M::L];
    gmx_operands<G>(x, A);
#pragma unroll 1
    for (int g = 0; g < J / 32 && t + 32 * g < need; g += 2) {
      const I4 B[2] = {coef[64 * g], coef[64 * (g + 1)]};
      // lane: step t + 32 g + lane
      if constexpr (M::S == 32) {
        uint32_t w[2];
#pragma unroll
        for (int i = 0; i < 2; i++) {
          const F16 c = gmx_chain<G>(A, B[i], offset);
          constexpr uint32_t digit = M::TOP ? 0x40404040u : 0x80808080u;
          uint32_t v = gmx_bytes<G>(c, 3);
          v = gmx_select(gmx_bytes<G>(c, 2), v >> 1, digit);
          v = gmx_select(gmx_bytes<G>(c, 1), v >> 1, digit);
          w[i] = gmx_select(gmx_bytes<G>(c, 0), v >> 1, digit);
        }
        const Swapped s = gmx_swap(w[0], w[1]);
        const uint64_t i = t + 32 * g + lane;
        const uint32_t word =
            M::TOP ? gmx_select(s.a << 1, s.b >> 3, 0xF0F0F0F0u) : gmx_select(s.a, s.b >> 4, 0xF0F0F0F0u);
        if (i < total) gmx_put<DT>(mine.out, i, word, dtype);
      } else if constexpr (M::S == 8) {
        uint32_t w[2][4];
#pragma unroll
        for (int i = 0; i < 2; i++) {
          const F16 c = gmx_chain<G>(A, B[i], offset);
#pragma unroll
          for (int k = 0; k < 4; k++) w[i][k] = gmx_bytes<G>(c, k);
        }
        uint64_t i = t + 32 * g + lane;
        // GQ58.4, and kernels of every type: no address of each stream (and
        // type) is kept across turns
        if constexpr (G == 7 || DT == kAnyType) asm volatile("" : "+v"(i));
#pragma unroll
        for (int k = 0; k < 4; k++) {
          const Swapped s = gmx_swap(w[0][k], w[1][k]);
          w[0][k] = M::TOP ? gmx_select(s.a << 4, s.b, 0xF0F0F0F0u) : gmx_select(s.a, s.b >> 4, 0xF0F0F0F0u);
        }
        if (DT != kAnyType || dtype != PRAND_F64) {
#pragma unroll
          for (int k = 0; k < 4; k++) {
            const GmxSec o = sec(k);
            if (i < o.n) gmx_put<DT>(o.out, i, w[0][k], dtype);
          }
        } else {
#pragma unroll
          for (int k = 0; k < 4; k++) {
            const GmxSec o = sec(k);
            if (i < o.n) put<PRAND_F64>(o.out, i, w[0][k]);
          }
        }
      } else {
        uint32_t w[2][2];
#pragma unroll
        for (int i = 0; i < 2; i++) {
          const F16 c = gmx_chain<G>(A, B[i], offset);
#pragma unroll
          for (int k = 0; k < 2; k++)
            w[i][k] = (gmx_pack3(gmx_bytes<G>(c, 2 * k)) << 12) | gmx_pack3(gmx_bytes<G>(c, 2 * k + 1));
        }
#pragma unroll
        for (int k = 0; k < 2; k++) {
          const Swapped s = gmx_swap(w[0][k], w[1][k]);
          // the step's 36 bits: elements 0-3, 4-7, 8-11
          const uint64_t chunk = ((uint64_t)(s.a >> 12) << 24) | (s.b & 0xFFF000u) | (s.a & 0xFFFu);
          // step 8 b + r starts 4 r bits into word 9 b + r: its top 32 - 4 r
          // bits end that word, the rest begin the next one
          const int r4 = 4 * (lane & 7);
          const uint32_t end = (uint32_t)(chunk >> (4 + r4)), begin = (uint32_t)(chunk << (28 - r4));
          const uint32_t prev = __builtin_amdgcn_update_dpp(0u, begin, 0x111, 0xf, 0xf, false);   // lane - 1
          uint64_t o0, tot;
          frame_of(k, o0, tot);
          char* const out = sec(k).out;
          const uint64_t i = (t + 32 * g) / 8 * 9 + lane + (lane >> 3);
          if (i >= o0 && i < tot) gmx_put<DT>(out, i - o0, r4 ? (prev | end) : end, dtype);
          if (r4 == 28 && i + 1 >= o0 && i + 1 < tot) gmx_put<DT>(out, i + 1 - o0, begin, dtype);
        }
      }
    }
    // move on: J steps, or to the output state
    const uint64_t left = save_at > t ? save_at - t : 0;
    uint64_t m0 = mj0, m1 = mj1;
    if (!__all(!live || left >= (uint64_t)J)) {
      const uint64_t* row = mats + 4 * (left < (uint64_t)J ? left : (uint64_t)J) + (upper ? 2 : 0);
      m0 = row[0];
      m1 = row[1];
    }
    uint64_t lower_x, upper_x;
    gmx_both(x, lower_x, upper_x);
    x = gmx_mulsum<G>(m0, lower_x, m1, upper_x);
  }
  gmx_round<false>();
  if (sout && !saved) save(x << M::T);
}

}  // namespace gm
}  // namespace prand
