// MT19937 on gfx950.
//
// Generation: one wavefront per stream, the 624-word state in LDS.  A twist
// renews the block in three dependency phases (words 0..226 read old words
// 397..623; 227..453 read words renewed in phase one; 454..623 read phase two
// and word 0), each phase parallel across the 64 lanes; whole blocks are
// written out two at a time from LDS as 16-byte pieces (dev_mt.h).  Where the
// streams are too few to fill the chip so, a workgroup of four wavefronts per
// stream makes 227 words at a time.
//
// Jump-ahead (paper, section on MT19937 jump-ahead, equation g_v):
// A^v Y = g_v(A) Y = sum_i a_i A^(i-1) Y with g_v = x^v mod phi.  A^(i-1) Y is
// the window of 624 consecutive raw words starting i-1 words later, so word t
// of the result is the XOR of seq[i + t] over the set coefficients i, seq
// being the raw-word sequence continued from the state.  A distance is applied
// as one polynomial x^(2^b) mod phi (from the context ladder) per set bit b;
// sections on block boundaries start by x^(d 624 2^(8 + 4 j)) mod phi per
// nonzero hexadecimal digit d of their distance in units of 2^8 blocks;
// block splitting by id * 2^432 from a block-aligned state uses the context's
// digit tables x^(d 2^(432 + position)) mod phi instead: three 16-bit digits
// for the low 48 bits of the id and two bytes for the top 16 bits; from the
// default state the top 16 bits come from a table of precomputed states, so a
// stream costs at most 3 polynomials.
// A workgroup of 4, 8 or 16 wavefronts does one stream: it produces the
// sequence into LDS, and each wavefront scans its own part of the
// coefficients: lane l accumulates outputs t = 10l .. 10l+9 while a register
// window of 10 sequence words slides over the coefficients, so each
// coefficient costs one LDS read per lane and set coefficients cost 10
// three-input XORs per two.  The partial windows are XORed at the end.
#include "dev_mt.h"
#include "mt_poly.h"
#include "prand_batch.h"

namespace prand {
namespace {

using namespace mt;


// Workgroup b (one wavefront) takes stream (b % 8) * (G / 8) + b / 8 for
// b < 8 (G / 8), G = count, else stream b: consecutive workgroups go to the
// eight XCDs in turn, so each XCD's L2 writes one contiguous eighth of the
// output (measured about 2 % faster than stream b).
template <int DT>
__global__ void __launch_bounds__(64) mt_generate_kernel(MtState* states, uint32_t count, uint64_t n,
                                                         void* __restrict__ out) {
  __shared__ __align__(16) uint32_t mt[2 * 624];
  const uint32_t b = blockIdx.x, per = count / 8;
  const uint32_t s = b < 8 * per ? (b % 8) * per + b / 8 : b;
  if (s >= count) return;
  constexpr int es = (DT == PRAND_F64) ? 8 : 4;
  gen_wave<DT>(mt, states + s, states + s, n, (char*)out + (uint64_t)s * n * es);
}

// a workgroup per stream (dev_mt.h)
template <int DT>
__global__ void __launch_bounds__(kGroup) mt_generate_group_kernel(MtState* states, uint64_t n, void* __restrict__ out) {
  __shared__ uint32_t ring[kRing];
  constexpr int es = (DT == PRAND_F64) ? 8 : 4;
  const uint32_t s = blockIdx.x;
  gen_group<DT>(ring, states + s, states + s, n, (char*)out + (uint64_t)s * n * es);
}

// sections of one stream, a workgroup each: section 0 starts from *base and has
// `first` outputs, section j from states[j - 1] and has seclen, the last one
// the rest; the state after it goes to *last
template <int DT>
__global__ void __launch_bounds__(kGroup) mt_sections_kernel(const MtState* base, const MtState* states, MtState* last,
                                                             uint64_t first, uint64_t seclen, uint64_t n,
                                                             void* __restrict__ out) {
  __shared__ uint32_t ring[kRing];
  constexpr int es = (DT == PRAND_F64) ? 8 : 4;
  const uint32_t j = blockIdx.x;
  const bool end = j + 1 == gridDim.x;
  const uint64_t start = j ? first + (j - 1) * seclen : 0;
  gen_group<DT>(ring, j ? states + (j - 1) : base, end ? last : nullptr, end ? n - start : (j ? seclen : first),
                (char*)out + start * es);
}

// Streams up to which a workgroup each is faster than a wavefront each, us for
// 100000 u32 / f64 per stream:
//   streams       1      256      512     1000     1500     2048
//   wavefront   98/106  104/113  113/124  113/169  141/259  189/326
//   workgroup   40/45    46/50    48/89    96/167  145/243  180/320
// (8192 streams of 20000 u32: 153 and 170; 65536 of 16384: 909 and 1080).
constexpr uint32_t kMtGroupMaxCount = 1024;

// ------------------------------------------------------------------ jump
// Wavefronts per stream by the launch's streams, all measured for block
// splitting from the default state (three polynomials; us):
//   streams      1   256   512  1000  2048  4096  8192  20000  65536
//   16         119   138   190   350   656  1283  2479   6563  19700
//   8          179   194   228   318   606  1167  2272   5823  18300
//   4          335   339   347   372   640  1183  2266   5518  17820
// (one wavefront per stream with an LDS ring of its own, the former form for
// more than 2048 streams, took 1231 us for one and 19300 us for 65536; its
// split forms, in which every wavefront ran the recurrence by itself up to its
// coefficients, 244 us for one stream and 639 us for 1000).
constexpr uint32_t kMtSplit16MaxCount = 512;
constexpr uint32_t kMtSplit8MaxCount = 4096;
constexpr int kDeg = 19937;
constexpr int kPer = 10;                    // outputs per lane: 64 * 10 >= 624

// s_waitcnt lgkmcnt(3), the other counters left at their maximum (gfx9
// encoding: vmcnt in bits 3:0 and 15:14, expcnt 6:4, lgkmcnt 11:8).
__device__ __forceinline__ void wait_lds_but3() { __builtin_amdgcn_s_waitcnt(0xC37F); }

// buf[0..623] holds a window (next output = tempered successor); apply_poly
// replaces it by g(A) applied to it, g = poly (624 words of coefficient bits,
// reduced: no bit at or above 19937 is set).  Lane l accumulates outputs
// t = 10 l + r.  For the coefficients i0 .. i0 + 9 of a group it holds the
// sequence words seq[i0 + 10 l + k] (cur) and seq[i0 + 10 + 10 l + k] (nxt),
// k < 10: coefficient i0 + u adds seq[i0 + u + 10 l + r], which is
// cur[u + r] or nxt[u + r - 10].  Three register windows rotate over the
// groups: while a group runs, the window the group after next starts with
// is read from LDS (pf), so no group waits for its own LDS reads.
//
// The coefficient bits are uniform across the wavefront, so the scan over
// them is scalar branching.  Each bit is tested once; a set bit waits for the
// next set bit of its group and the two are added with one three-input XOR
// (gfx950 v_bitop3_b32, truth table 0x96) per output word: a group with c set
// coefficients costs ceil(c / 2) instead of c vector instructions per output
// word.  The scan is a chain of labels joined by gotos (mt_pairs.inc; after a
// pair the remaining nothing-pending tests are repeated in place, one taken
// branch less per pair), built with the structurizer told to leave uniform
// regions alone, so every test is one scalar compare and branch.
// i0 is counted from the buffer's first word.
template <int kOff>
__device__ __forceinline__ void group(const uint32_t* buf, uint32_t i0, uint32_t lo, uint32_t hi, int lane,
                                      uint32_t (&acc)[kPer],
                                      const uint32_t (&cur)[kPer], const uint32_t (&nxt)[kPer],
                                      uint32_t (&pf)[kPer]) {
  // i0 + 20 + 10 lane is even, so the window is read in 8-byte pairs
  const uint32_t* src = buf + ((i0 + 2 * kPer + kPer * lane) & ~1u);
#pragma unroll
  for (int k = 0; k < kPer; k++) pf[k] = src[k];
  // the window nxt was read by the previous group: wait for those reads once
  // here (the three just issued may stay in flight), not before every pair
  wait_lds_but3();
#define MT_W2(k) (((k) < kPer) ? cur[(k)] : nxt[(k) - kPer])
#define MT_BIT(u) (((kOff + (u)) < 32 ? (lo >> ((kOff + (u)) & 31)) : (hi >> ((kOff + (u)) & 31))) & 1u)
#define MT_PAIR(p, q)                                                                              \
  _Pragma("unroll") for (int r = 0; r < kPer; r++) acc[r] =                                        \
      __builtin_amdgcn_bitop3_b32(acc[r], MT_W2((p) + r), MT_W2((q) + r), 0x96);
#define MT_ONE(p) _Pragma("unroll") for (int r = 0; r < kPer; r++) acc[r] ^= MT_W2((p) + r);
#include "mt_pairs.inc"
#undef MT_ONE
#undef MT_PAIR
#undef MT_BIT
#undef MT_W2
}

// Coefficients are scanned 60 at a time (six groups), each group testing its
// bits at fixed positions of two 32-bit scalar words (bits i1 .. i1 + 63).
// The three polynomial words a step needs are read one step ahead through
// the vector memory path, as a 624-word raw buffer (the byte offset in a
// vector register, so the hardware range check covers it: a word past the
// polynomial reads as zero), then moved to scalar registers.  Scalar loads
// would share the LDS wait counter and, returning out of order, force a full
// wait before every pair of a step.  Measured 3.4 % faster than scalar loads
// with masked group bits.  Also measured: the next window moved across lanes
// by DPP wavefront shifts, with only the last lane reading the ring, 4 %
// slower; the LDS reads are not the limit, the chain of scalar tests and
// branches of each wavefront is.
constexpr uint32_t kStep = 6 * kPer;
constexpr int kStepReach = 720;   // a step at i1 reads sequence words below i1 + 710

typedef __amdgpu_buffer_rsrc_t PolyBuf;

__device__ __forceinline__ PolyBuf poly_buffer(const uint32_t* poly) {
  // gfx9 buffer descriptor: base, no stride, 624 * 4 bytes, 32-bit data format
  return __builtin_amdgcn_make_buffer_rsrc((void*)poly, 0, 624 * 4, 0x00020000);
}

__device__ __forceinline__ uint32_t poly_word(PolyBuf pb, uint32_t w) {
  uint32_t off = w * 4u;
  asm volatile("" : "+v"(off));   // the whole offset in the vector operand
  return __builtin_amdgcn_raw_buffer_load_b32(pb, off, 0, 0);
}

// apply_poly by the kParts wavefronts of a workgroup: the sequence is
// produced by all of them, segment by segment into a linear LDS buffer; of a
// segment's coefficients each wavefront scans its own kChunk (a multiple of
// kStep), and at the end the partial sums, which add up to the whole because
// g(A) Y is linear in the coefficients, are XORed together through LDS.
// Segments: as few as leave eight wavefronts per SIMD (4 and 8 parts: 19 and
// 31 KB per workgroup); fewer or more measured 1-5 % slower.
template <int kParts>
struct Split {
  static constexpr int kThreads = 64 * kParts;
  static constexpr uint32_t kSegs = kParts == 4 ? 6 : 3;
  static constexpr uint32_t kChunk = ((kDeg + kParts * kSegs - 1) / (kParts * kSegs) + kStep - 1) / kStep * kStep;
  static constexpr uint32_t kSeg = kChunk * kParts;               // coefficients of a segment
  static constexpr int kPhase = kThreads < 623 ? kThreads : 623;   // words a phase adds
  static constexpr int kHold = (int)kSeg + kStepReach + kPhase;
  static constexpr int kSum = 640 * kParts;
  static constexpr int kLds = kHold > kSum ? kHold : kSum;        // words
  static constexpr int kWords = (624 + kThreads - 1) / kThreads;   // combined words per thread
  static_assert(kSeg * kSegs >= (uint32_t)kDeg, "the segments cover the polynomial");
  static_assert(kSeg >= (uint32_t)(kStepReach + kPhase), "a segment's words past its end move without overlap");
};

// words that the recurrence takes from the pair (x_j, x_{j+1})
__device__ __forceinline__ uint32_t twist_pair(const uint32_t* x) { return recur(x[0], x[1], 0); }

// Extend buf[0 .. have) (have >= 624 words of the sequence) to at least
// `need` words, kPhase words at a time: word have + t is x_{j+397} + the pair
// of x_j (j = have - 624 + t), and where x_{j+397} is itself new (t >= 227,
// again from t >= 454), the recurrence is put in for it, so a phase needs no
// word of its own and one barrier serves up to 623 words instead of 227.
template <int kParts>
__device__ __forceinline__ void extend_shared(uint32_t* buf, int& have, int need) {
  const int t = (int)threadIdx.x;
  while (have < need) {
    if (t < Split<kParts>::kPhase) {
      const uint32_t* x = buf + have - 624 + t;
      uint32_t v = twist_pair(x);
      if (t < 227) {
        v ^= x[397];
      } else if (t < 454) {
        v ^= x[170] ^ twist_pair(x - 227);
      } else {
        v ^= x[-57] ^ twist_pair(x - 227) ^ twist_pair(x - 454);
      }
      buf[have + t] = v;
    }
    have += Split<kParts>::kPhase;
    __syncthreads();
  }
}

// The sum over the coefficients c0 <= i < c1 of poly added to sum (lane l
// holds outputs t = 10 l + r); buf[0] is word `base` of the sequence, c0 and
// base multiples of kStep, c1 one too or kDeg
__device__ __forceinline__ void scan(const uint32_t* buf, const uint32_t* __restrict__ poly, int lane, uint32_t c0,
                                            uint32_t c1, uint32_t base, uint32_t (&sum)[kPer]) {
  // acc is local: the groups' code is built on a register array
  uint32_t acc[kPer], wa[kPer], wb[kPer], wc[kPer];
  // the first two windows, read as group() reads the later ones
  const uint32_t* w0 = buf + ((c0 - base + kPer * lane) & ~1u);
#pragma unroll
  for (int r = 0; r < kPer; r++) {
    acc[r] = sum[r];
    wa[r] = w0[r];
    wb[r] = w0[kPer + r];
  }
  // bits i1 .. i1 + 59 lie in the words i1 / 32 .. i1 / 32 + 2 (the last
  // step's third word is past the polynomial and reads as zero)
  const PolyBuf pb = poly_buffer(poly);
  uint32_t n0 = poly_word(pb, c0 >> 5), n1 = poly_word(pb, (c0 >> 5) + 1), n2 = poly_word(pb, (c0 >> 5) + 2);
  for (uint32_t i1 = c0; i1 < c1; i1 += kStep) {
    const uint32_t p0 = __builtin_amdgcn_readfirstlane(n0), p1 = __builtin_amdgcn_readfirstlane(n1),
                   p2 = __builtin_amdgcn_readfirstlane(n2);
    const uint32_t wn = (i1 + kStep) >> 5;
    n0 = poly_word(pb, wn);
    n1 = poly_word(pb, wn + 1);
    n2 = poly_word(pb, wn + 2);
    const uint32_t sh = i1 & 31;
    uint32_t b0 = (uint32_t)((((uint64_t)p1 << 32) | p0) >> sh);
    uint32_t b1 = (uint32_t)((((uint64_t)p2 << 32) | p1) >> sh);
    asm volatile("" : "+s"(b0), "+s"(b1));   // every test reads these two words
    const uint32_t i0 = i1 - base;
    group<0>(buf, i0, b0, b1, lane, acc, wa, wb, wc);
    group<kPer>(buf, i0 + kPer, b0, b1, lane, acc, wb, wc, wa);
    group<2 * kPer>(buf, i0 + 2 * kPer, b0, b1, lane, acc, wc, wa, wb);
    group<3 * kPer>(buf, i0 + 3 * kPer, b0, b1, lane, acc, wa, wb, wc);
    group<4 * kPer>(buf, i0 + 4 * kPer, b0, b1, lane, acc, wb, wc, wa);
    group<5 * kPer>(buf, i0 + 5 * kPer, b0, b1, lane, acc, wc, wa, wb);
  }
#pragma unroll
  for (int r = 0; r < kPer; r++) sum[r] = acc[r];
}

// buf[0 .. 624) holds the window; every thread of the workgroup calls, with
// the window in place for all of them
template <int kParts>
__device__ __forceinline__ void apply_poly(uint32_t* buf, const uint32_t* __restrict__ poly, int lane, int part) {
  using S = Split<kParts>;
  uint32_t sum[kPer];
#pragma unroll
  for (int r = 0; r < kPer; r++) sum[r] = 0;
  int have = 624;
#pragma unroll 1
  for (uint32_t g = 0; g < S::kSegs; g++) {
    const uint32_t base = g * S::kSeg;
    if (g) {
      // the words past the segment move to the front (fewer than kSeg)
      have -= (int)S::kSeg;
      for (int i = (int)threadIdx.x; i < have; i += S::kThreads) buf[i] = buf[S::kSeg + i];
      __syncthreads();
    }
    extend_shared<kParts>(buf, have, (int)S::kSeg + kStepReach);
    const uint32_t c0 = base + (uint32_t)part * S::kChunk;
    const uint32_t c1 = c0 + S::kChunk < (uint32_t)kDeg ? c0 + S::kChunk : (uint32_t)kDeg;
    if (c0 < c1) scan(buf, poly, lane, c0, c1, base, sum);
    __syncthreads();   // the segment's words are read
  }
#pragma unroll
  for (int r = 0; r < kPer; r++) buf[640 * part + kPer * lane + r] = sum[r];
  __syncthreads();   // every partial sum in place
  uint32_t v[S::kWords];
#pragma unroll
  for (int k = 0; k < S::kWords; k++) {
    const int t = (int)threadIdx.x + S::kThreads * k;
    v[k] = 0;
    if (t < 624) {
#pragma unroll
      for (int p = 0; p < kParts; p++) v[k] ^= buf[640 * p + t];
      if (t == 0) v[k] &= kUpper;
    }
  }
  __syncthreads();   // every partial sum read
#pragma unroll
  for (int k = 0; k < S::kWords; k++) {
    const int t = (int)threadIdx.x + S::kThreads * k;
    if (t < 624) buf[t] = v[k];
  }
  __syncthreads();
}

// Lowest set bit of the multi-limb number N at or above bit `from`, or -1.
__device__ __forceinline__ int next_bit(const uint64_t (&N)[kMaxLimbs], int from) {
#pragma unroll
  for (int l = 0; l < kMaxLimbs; l++) {
    if (from < 64 * (l + 1)) {
      uint64_t w = N[l];
      if (from > 64 * l) w &= ~0ull << (from - 64 * l);
      if (w) return 64 * l + __builtin_ctzll(w);
    }
  }
  return -1;
}

// A workgroup of kParts wavefronts per stream.
template <int kParts>
__global__ void __launch_bounds__(64 * kParts) mt_jump_kernel(MtState* __restrict__ states, uint32_t count,
                                                     const uint64_t* __restrict__ dist, int nlimbs, int per_stream,
                                                     const uint64_t* __restrict__ ids, int block_e,
                                                     const MtState* __restrict__ base,
                                                     const MtState* __restrict__ top,
                                                     const uint32_t* __restrict__ ladder,
                                                     const uint32_t* __restrict__ diglo,
                                                     const uint32_t* __restrict__ dig8hi,
                                                     const uint32_t* __restrict__ blk, int blocks) {
  __shared__ __align__(16) uint32_t buf[Split<kParts>::kLds];
  const uint32_t s = blockIdx.x;
  if (s >= count) return;
  // the scan is one long chain of dependent scalar tests and branches: where
  // its wavefronts share a SIMD with other kernels' (a served stream start
  // beside generation chunks), the highest wave priority lets the chain
  // issue first instead of waiting behind the others' VALU work
  __builtin_amdgcn_s_setprio(3);
  const int lane = threadIdx.x & 63;
  // the wavefront's part, uniform across it (its coefficient range is scanned
  // by scalar branching)
  const int part = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  // block splitting from the default state: start from the precomputed
  // state of the id's top 16 bits
  const bool digit_path = ids && block_e == kMtDigitE;
  const MtState* src = base ? base : states + s;
  if (digit_path && top) src = top + (ids[s] >> 48);
  uint64_t N[kMaxLimbs];
  for (int l = 0; l < kMaxLimbs; l++) N[l] = 0;
  if (ids) {
    const uint64_t id = ids[s];
    const int q = block_e >> 6, r = block_e & 63;
    N[q] = id << r;
    if (r && q + 1 < kMaxLimbs) N[q + 1] = id >> (64 - r);
  } else {
    const uint64_t* d = dist + (per_stream ? (size_t)s * nlimbs : 0);
    for (int l = 0; l < nlimbs; l++) N[l] = d[l];
  }
  for (int i = (int)threadIdx.x; i < 624; i += 64 * kParts) buf[i] = src->mt[i];
  uint32_t idx = src->idx < 624u ? src->idx : 624u;
  __syncthreads();
  // the polynomials to apply, in order: for block splitting from a
  // block-aligned state, id * 2^432 with the low 48 bits of id as 16-bit
  // digits and the top 16 bits as two bytes, one table polynomial
  // x^(d 2^(432 + position)) per nonzero digit (the top bytes are already in
  // the start state when it came from the table of top-16-bit states);
  // otherwise one ladder polynomial x^(2^b) per set bit b of the distance
  // left after the rest of the current block.  One call site keeps a single
  // copy of the polynomial code.
  const bool use_digits = digit_path && idx == 624;
  const uint64_t id = ids ? ids[s] : 0;
  // distances D in whole sections: from a block boundary, and D within the
  // table, one whole-block polynomial per nonzero hexadecimal digit of the
  // distance in units (the state stays on a boundary); otherwise the distance
  // in outputs, D (624 2^kMtBlkFirst), through the ladder
  if (blocks == kMtUnits) idx = 624;
  const bool sec_units = blocks == kMtSections && !ids;
  const bool use_blocks = blocks == kMtUnits || (sec_units && idx == 624 && (N[0] >> kMtBlkPolys) == 0);
  if (sec_units && use_blocks) N[0] <<= kMtBlkFirst - kMtBlkUnit;
  if (sec_units && !use_blocks) {
    constexpr uint64_t kSec = 624ull << kMtBlkFirst;
    const uint64_t d = N[0];
    N[0] = d * kSec;
    N[1] = __umul64hi(d, kSec);
  }
  if (!use_digits && !use_blocks) {
    const uint64_t rest = 624 - idx;
    bool small = true;
    for (int l = 1; l < kMaxLimbs; l++) small = small && (N[l] == 0);
    small = small && (N[0] <= rest);
    if (small) {
      idx += (uint32_t)N[0];
      for (int l = 0; l < kMaxLimbs; l++) N[l] = 0;
    } else {
      uint64_t borrow = rest;
      for (int l = 0; l < kMaxLimbs && borrow; l++) {
        const uint64_t old = N[l];
        N[l] = old - borrow;
        borrow = old < borrow ? 1 : 0;
      }
      idx = 624;
    }
  }
  const int ndig = top ? kMtLoDigits : kMtLoDigits + 2;
  int pos = 0;
  for (;;) {
    const uint32_t* poly = nullptr;
    if (use_digits) {
      for (; pos < ndig && !poly; pos++) {
        if (pos < kMtLoDigits) {
          const uint32_t d = (uint32_t)(id >> (kMtLoBits * pos)) & (uint32_t)(kMtLoSize - 1);
          if (d) poly = diglo + ((size_t)pos * kMtLoSize + d) * 624;
        } else {
          const int j = pos - kMtLoDigits;
          const uint32_t d = (uint32_t)(id >> (48 + 8 * j)) & 255u;
          if (d) poly = dig8hi + ((size_t)j * 256 + d) * 624;
        }
      }
    } else if (use_blocks) {
      for (; pos < kMtBlkDigits && !poly; pos++) {
        const uint32_t d = (uint32_t)(N[0] >> (4 * pos)) & 15u;
        if (d) poly = blk + ((size_t)pos * 16 + d) * 624;
      }
    } else {
      const int b = next_bit(N, pos);
      if (b >= 0) {
        poly = ladder + (size_t)b * 624;
        pos = b + 1;
      }
    }
    if (!poly) break;
    apply_poly<kParts>(buf, poly, lane, part);
  }
  MtState* dst = states + s;
  for (int i = (int)threadIdx.x; i < 624; i += 64 * kParts) dst->mt[i] = buf[i];
  if (threadIdx.x == 0) {
    dst->idx = idx;
    dst->pad[0] = dst->pad[1] = dst->pad[2] = 0;
  }
}

// Start state of an MT19937 section tile of a batch: the task state moved
// D = first * kMtSection outputs on, a whole number of 624-word blocks, so
// the state keeps the task's block grid and its place in the block (idx)
// and equals the state sequential generation would reach.  x^D (one
// whole-block polynomial per nonzero digit of the distance) moves
// every word of the array D places along the sequence but leaves only the
// top bit of the oldest word exact; x^(-1) then steps the window one word
// back, so that the array's words 1..623 are the exact words 0..622 of the
// target window, and one step of the recurrence supplies its word 623.
// Section 0 is a copy.
constexpr int kSectionParts = 8;

__global__ void __launch_bounds__(64 * kSectionParts)
    mt_section_start_kernel(const BatchTile* __restrict__ tiles, uint32_t ntiles, const BatchTask* __restrict__ tasks,
                            char* __restrict__ scratch, const uint32_t* __restrict__ blk,
                            const uint32_t* __restrict__ inv) {
  __shared__ __align__(16) uint32_t buf[Split<kSectionParts>::kLds];
  const uint32_t t = blockIdx.x;
  if (t >= ntiles) return;
  const BatchTile tl = tiles[t];
  if (tl.kind != kTileMtSection) return;
  const int lane = threadIdx.x & 63;
  const int part = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const MtState* src = (const MtState*)tasks[tl.task].state_in;
  MtState* dst = (MtState*)(scratch + tl.starts);
  for (int i = (int)threadIdx.x; i < 624; i += 64 * kSectionParts) buf[i] = src->mt[i];
  const uint32_t idx = src->idx < 624u ? src->idx : 624u;
  __syncthreads();
  if (tl.first == 0) {
    for (int i = (int)threadIdx.x; i < 624; i += 64 * kSectionParts) dst->mt[i] = buf[i];
  } else {
    // one polynomial per nonzero digit of the distance in units, then x^(-1)
    const uint64_t units = tl.first << (kMtBlkFirst - kMtBlkUnit);
    for (int k = 0; k <= kMtBlkDigits; k++) {
      const uint32_t d = k < kMtBlkDigits ? (uint32_t)(units >> (4 * k)) & 15u : 1u;
      if (d) apply_poly<kSectionParts>(buf, k < kMtBlkDigits ? blk + ((size_t)k * 16 + d) * 624 : inv, lane, part);
    }
    for (int i = (int)threadIdx.x; i < 623; i += 64 * kSectionParts) dst->mt[i] = buf[i + 1];
    if (threadIdx.x == 0) dst->mt[623] = recur(buf[0], buf[1], buf[397]);
  }
  if (threadIdx.x == 0) {
    dst->idx = idx;
    dst->pad[0] = dst->pad[1] = dst->pad[2] = 0;
  }
}

}  // namespace

hipError_t launch_batch_mt_starts(const DeviceTables& T, const BatchTile* tiles, uint32_t ntiles,
                                  const BatchTask* tasks, char* scratch, hipStream_t st) {
  return launch_ranges(ntiles, 64 * kSectionParts, 1, [&](uint64_t first, uint32_t m, uint32_t blocks) {
    hipLaunchKernelGGL(mt_section_start_kernel, dim3(blocks), dim3(64 * kSectionParts), 0, st, tiles + first, m, tasks,
                       scratch, T.mtblk, T.mtinv);
    return hipGetLastError();
  });
}

hipError_t launch_mt_generate(MtState* states, uint32_t count, uint64_t n, int dtype, void* out, hipStream_t st) {
  if (count <= kMtGroupMaxCount) {
    const dim3 grid(count), block(kGroup);
    switch (dtype) {
      case PRAND_U32: hipLaunchKernelGGL(mt_generate_group_kernel<PRAND_U32>, grid, block, 0, st, states, n, out); break;
      case PRAND_F32: hipLaunchKernelGGL(mt_generate_group_kernel<PRAND_F32>, grid, block, 0, st, states, n, out); break;
      default: hipLaunchKernelGGL(mt_generate_group_kernel<PRAND_F64>, grid, block, 0, st, states, n, out); break;
    }
    return hipGetLastError();
  }
  return launch_ranges(count, 64, 1, [&](uint64_t first, uint32_t m, uint32_t blocks) {
    const dim3 grid(blocks), block(64);
    MtState* const s = states + first;
    char* const o = (char*)out + first * n * (dtype == PRAND_F64 ? 8 : 4);
    switch (dtype) {
      case PRAND_U32: hipLaunchKernelGGL(mt_generate_kernel<PRAND_U32>, grid, block, 0, st, s, m, n, o); break;
      case PRAND_F32: hipLaunchKernelGGL(mt_generate_kernel<PRAND_F32>, grid, block, 0, st, s, m, n, o); break;
      default: hipLaunchKernelGGL(mt_generate_kernel<PRAND_F64>, grid, block, 0, st, s, m, n, o); break;
    }
    return hipGetLastError();
  });
}

hipError_t launch_mt_sections(const MtState* base, const MtState* states, MtState* last, uint32_t count, uint64_t first,
                              uint64_t seclen, uint64_t n, int dtype, void* out, hipStream_t st) {
  const dim3 grid(count), block(kGroup);
  switch (dtype) {
    case PRAND_U32:
      hipLaunchKernelGGL(mt_sections_kernel<PRAND_U32>, grid, block, 0, st, base, states, last, first, seclen, n, out);
      break;
    case PRAND_F32:
      hipLaunchKernelGGL(mt_sections_kernel<PRAND_F32>, grid, block, 0, st, base, states, last, first, seclen, n, out);
      break;
    default:
      hipLaunchKernelGGL(mt_sections_kernel<PRAND_F64>, grid, block, 0, st, base, states, last, first, seclen, n, out);
      break;
  }
  return hipGetLastError();
}

hipError_t launch_mt_jump(const DeviceTables& T, MtState* states, uint32_t count, const JumpSpec& js,
                          const MtState* base, hipStream_t st) {
  // whole-section distances: one limb per stream
  if (js.mt_blocks && (js.ids || !js.per_stream || js.nlimbs != 1)) return hipErrorInvalidValue;
  const uint32_t parts = count <= kMtSplit16MaxCount ? 16 : count <= kMtSplit8MaxCount ? 8 : 4;
  return launch_ranges(count, 64 * parts, 1, [&](uint64_t first, uint32_t m, uint32_t blocks) {
    auto launch = [&](auto* kernel) {
      hipLaunchKernelGGL(kernel, dim3(blocks), dim3(64 * parts), 0, st, states + first, m,
                         js.per_stream ? js.dist + first * js.nlimbs : js.dist, js.nlimbs, js.per_stream,
                         js.ids ? js.ids + first : nullptr, js.block_e, base, (const MtState*)js.mt_top, T.mt, T.mtdiglo,
                         T.mtdig8hi, T.mtblk, js.mt_blocks);
      return hipGetLastError();
    };
    return parts == 16 ? launch(mt_jump_kernel<16>) : parts == 8 ? launch(mt_jump_kernel<8>) : launch(mt_jump_kernel<4>);
  });
}

}  // namespace prand
