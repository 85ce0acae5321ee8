// GM19, GM29, GM31, GM55, GM61, GQ58.1, GQ58.3, GQ58.4 on gfx950: ensembles of
// s torus maps x_i^(n) = k x_i^(n-1) - q x_i^(n-2) mod g (paper, equation
// rec1; k, q, g, v of Table 2).  Each element contributes a v-bit digit
// floor(2^v x / g) per step; digits are packed element 0 first, most
// significant bit first, into 32-bit words (GQ58.3: 36 bits per step, 9 words
// per 8 steps).
//
// Generation by matrix instructions (dev_gmx.h): a wavefront holds the 32
// elements of one v = 1 stream, or of four 8-element or two 12-element ones;
// short runs of the v = 1 ensembles keep one lane per element and one ballot
// per word (dev_gm.h).  Few streams are cut into sections that start by jumps.
//
// Arithmetic is exact.  For g = p 2^t (GM55: t = 4, GQ58: t = 29) the even
// k and q kill the 2-adic part within n0 steps; from then on x = 2^t y with y
// following the same recurrence mod p and the digit equal to
// floor(2^v y / p), so the kernels run exact mod-g steps only until every
// element of the wavefront has collapsed and then switch to the mod-p
// recurrence.
#include "dev_gm.h"
#include "dev_gmx.h"

namespace prand {
namespace {

using namespace gm;

// wavefronts that fill the chip (four to five per SIMD, twice over)
constexpr uint64_t kFillWaves = 8192;

// Short runs of a v = 1 ensemble: half a wavefront per stream, one lane per
// element, a ballot per word (dev_gm.h).  The matrix form makes the operands of
// 256 steps, turns of 64 steps, and moves the states by a product: 65536 GM29
// streams of 1, 32 and 100 outputs take 17, 29 and 61 us by ballots, 52, 52 and 71
// so.  From 128 outputs on it costs, in ballot outputs, a fixed part and parts per
// 256 steps and per turn, more where states and outputs are well beyond the
// memory-side cache (256 MB): it has half as many streams in a wavefront, waiting
// for their states.  Ballots where that is more than n: 65536 GM61 streams of 144 outputs
// 104 us (by the matrix form 116), of 192 134 (118); 300000 GM19 streams of 128 f64
// 169 (273), of 512 587 (640), of 800 964 (923).  (The v >= 3 ensembles are
// faster by the matrix form at any length: 65536 streams of 1, 32 and 128 u32,
// GM55 30, 40 and 69 us by a lane per section, 24, 25 and 31 so; GQ58.3 48, 54 and
// 88, 37, 39 and 51; GQ58.4 30, 38 and 55, 21, 22 and 26.)
struct BallotCost {
  uint32_t fixed, advance, turn;
};
struct BallotRule {
  BallotCost small, large, large64;   // 64: f64
};
template <int G>
bool ballots(uint64_t count, uint64_t n, uint64_t es) {
  static_assert(Mx<G>::S == 32, "a lane per element");
  constexpr BallotRule r = G == 0   ? BallotRule{{45, 15, 40}, {85, 0, 50}, {120, 0, 54}}
                           : G == 4 ? BallotRule{{18, 15, 43}, {45, 0, 47}, {60, 0, 45}}
                                    : BallotRule{{46, 0, 34}, {44, 0, 45}, {62, 0, 44}};
  if (n < 128) return true;
  if (n >= 1024 || count < 2 * kFillWaves) return false;
  const bool large = count * (2 * sizeof(GmState) + n * es) > (440u << 20);
  const BallotCost c = !large ? r.small : es == 8 ? r.large64 : r.large;
  return n < c.fixed + c.advance * ((n + 255) / 256) + c.turn * ((n + 63) / 64);
}

template <int G, int DT>
__global__ void __launch_bounds__(256) gm_gen32_kernel(const GmState* sin, GmState* sout, uint32_t count, uint64_t n,
                                                       void* __restrict__ out) {
  const uint64_t s = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 5;
  const bool live = s < count;
  constexpr int es = (DT == PRAND_F64) ? 8 : 4;
  gen32_wave<G, DT>(live, sin + (live ? s : 0), sout + (live ? s : 0), n, (char*)out + s * n * es);
}

// Many streams: a wavefront takes Mx<G>::Q consecutive (stream, section)
// pairs; the sections of a stream cover [j seclen, min((j + 1) seclen, n)).
// kSections: several sections per stream, which read the stream's state and
// jump to their starts; the states are then moved on by a launch of their own
// (sout null), or, of a single stream, the last section leaves the state in
// *sout (another object than *sin).  Otherwise seclen = n and the states are
// updated in place.
template <int G, int DT, bool kSections>
__global__ void __launch_bounds__(256) gmx_kernel(const GmState* sin, GmState* sout, uint32_t count, uint64_t n,
                                                  uint32_t nsec, uint64_t seclen, char* __restrict__ out,
                                                  const GmxTable* __restrict__ table,
                                                  const uint64_t* __restrict__ ladder) {
  constexpr int Q = Mx<G>::Q;
  constexpr int es = (DT == PRAND_F64) ? 8 : 4;
  __shared__ uint32_t lds[4][kGmxLds];
  const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint64_t first = ((uint64_t)blockIdx.x * 4 + w) * Q;
  const uint64_t all = kSections ? (uint64_t)count * nsec : count;
  if (first >= all) return;
  // one division, here: sec() is called in the generation loop too (with a
  // division per pair and turn left there and now: 300 GM55 streams of 20000 u32
  // 35 and 28 us, 10^7 GQ58.3 numbers of one state 86 and 75, 10^8 GQ58.4 226 and
  // 171).  In 64 bits, which the compiler branches around: by a 32-bit division
  // the v = 1 kernels came out with 4-20 registers more, GM61's a wavefront less
  const uint32_t s0 = kSections ? (uint32_t)(first / nsec) : 0;
  const uint32_t j0 = kSections ? (uint32_t)first - s0 * nsec : 0;   // (count nsec < 2^32: launch_gen)
  auto sec = [&](int q) {
    uint32_t s1 = s0, j = j0 + q;
    if (kSections) {
#pragma unroll
      for (int c = 1; c < Q; c++)
        if (c <= q && j >= nsec) {
          j -= nsec;
          s1++;
        }
    }
    const uint64_t s = kSections ? s1 : first + q, start = kSections ? j * seclen : 0;
    GmxSec r{nullptr, start, 0, nullptr, nullptr};
    if (first + q < all) {
      r.in = sin + s;
      r.n = kSections ? (n - start < seclen ? n - start : seclen) : n;
      r.out = out + (s * n + start) * es;
      r.sout = !kSections ? sout + s : (sout && start + r.n == n ? sout : nullptr);
    }
    return r;
  };
  gmx_wave<G, DT, kSections>(sec, table + G, ladder, lds[w]);
}

// lanes per stream of the jump: one per element; GQ58.3's twelve in a group of
// sixteen, so that a stream's lanes share a wavefront (all of them read the
// state's word offset before one of them writes it)
template <int G>
constexpr uint32_t jump_lanes() {
  return kGmParams[G].s == 12 ? 16 : kGmParams[G].s;
}

// One lane per element: states[s] = base (or states[s]) jumped by the
// stream's distance; GQ58.3 distances count words.  Block splitting with the
// default block exponent takes the byte tables (at most eight matrices per
// stream), other distances the ladder (one per set bit).  A state's unused
// element slots are left alone where it moves in place and copied from the
// base otherwise.  Bound: the modular products (GM55 and GM61: 128-bit) and the
// state lines.  (With a lane per slot, 32 per stream, a wavefront of the 8-
// and 12-element ensembles did its products with a quarter or a third of its
// lanes, and every slot was read and written; GQ58.3 took a matrix per set bit
// of its distance in elements.  2^20 states moved 2^k: GM55 494 -> 186 us,
// GQ58.4 363 -> 188, GQ58.3 1490 -> 361; started by block splitting: GM55
// 711 -> 236, GQ58.4 670 -> 220, GQ58.3 669 -> 369.)
template <int G>
__global__ void __launch_bounds__(256) gm_jump_kernel(GmState* __restrict__ states, uint32_t count,
                                                      const uint64_t* __restrict__ dist, int nlimbs, int per_stream,
                                                      uint64_t fixed, const uint64_t* __restrict__ ids, int block_e,
                                                      const GmState* __restrict__ base,
                                                      const uint64_t* __restrict__ ladder,
                                                      const uint64_t* __restrict__ bytetab,
                                                      const uint64_t* __restrict__ neg) {
  constexpr uint32_t S = kGmParams[G].s, kLanes = jump_lanes<G>();
  const uint64_t gid = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const uint64_t s = gid / kLanes;
  const uint32_t e = (uint32_t)(gid % kLanes);
  if (s >= count || e >= S) return;
  const GmState* src = base ? base : states + s;
  GmState* dst = states + s;
  uint64_t xc = src->xc[e], xp = src->xp[e];
  uint32_t off = (G == 6) ? src->off : 0;
  if (ids && bytetab && block_e == kGmByteE[G]) {
    // whole blocks: the offset inside a GQ58.3 block is kept
    jump_bytes_elem<G>(xc, xp, ids[s], bytetab, neg);
  } else {
    uint64_t N[kMaxLimbs + 1];
    for (int l = 0; l <= kMaxLimbs; l++) N[l] = 0;
    if (ids) {
      const uint64_t id = ids[s];
      const int q = block_e >> 6, r = block_e & 63;   // block in ensemble steps
      N[q] = id << r;
      if (r) N[q + 1] = id >> (64 - r);
    } else if (dist) {
      const uint64_t* d = dist + (per_stream ? (size_t)s * nlimbs : 0);
      for (int l = 0; l < nlimbs; l++) N[l] = d[l];
    } else {
      N[0] = fixed;
    }
    // whole blocks of an id keep the offset inside the block
    if (G == 6 && !ids) gq3_words_to_steps(N, off, &off);
    jump_steps_elem<G>(xc, xp, N, ladder);
  }
  dst->xc[e] = xc;
  dst->xp[e] = xp;
  if (base)
    for (uint32_t i = S + e; i < 32; i += S) {
      dst->xc[i] = base->xc[i];
      dst->xp[i] = base->xp[i];
    }
  if (e == 0) {
    dst->off = off;
    dst->pad = 0;
  }
}

template <int G>
hipError_t launch_jump_g(const DeviceTables& T, GmState* states, uint32_t count, const JumpSpec& js,
                         const GmState* base, hipStream_t st) {
  return launch_ranges(count, 256, 256 / jump_lanes<G>(), [&](uint64_t first, uint32_t m, uint32_t blocks) {
    hipLaunchKernelGGL(gm_jump_kernel<G>, dim3(blocks), dim3(256), 0, st, states + first, m,
                       js.per_stream ? js.dist + first * js.nlimbs : js.dist, js.nlimbs, js.per_stream, js.fixed,
                       js.ids ? js.ids + first : nullptr, js.block_e, base, T.gm,
                       T.gmbyte ? T.gmbyte + (size_t)G * 8 * 256 * 4 : nullptr,
                       T.gmneg ? T.gmneg + (size_t)G * 4 : nullptr);
    return hipGetLastError();
  });
}

// Sections per stream.  At least kFillWaves wavefronts of whole streams stay
// whole; fewer are cut into
// sections of whole state advances, as long as there stay enough of them: of
// eight advances (a section's start is one matrix per nonzero byte of its
// distance, about the time of two advances), or down to one where there would
// be less than a wavefront per SIMD, for streams of at least three (the states
// then move on by a launch of their own: 4 us.  196 GM55 streams of 5148 u32 in
// sections of eight advances 56 us, of one 20; 61 GM31 of 2792 36 us whole, 15
// so; 100 GM61 of 1000 24 and 16)
template <int G, int DT>
hipError_t launch_gen(const DeviceTables& T, GmState* states, uint32_t count, uint64_t n, void* out, hipStream_t st) {
  constexpr uint64_t Q = Mx<G>::Q, es = DT == PRAND_F64 ? 8 : 4;
  constexpr uint64_t unit = G == 6 ? kGmxSteps / 8 * 9 : kGmxSteps;   // outputs of a state advance
  uint64_t seclen = 8 * unit;
  if constexpr (Mx<G>::S == 32) {
    if (ballots<G>(count, n, es)) {
      return launch_ranges(count, 256, 8, [&](uint64_t first, uint32_t m, uint32_t blocks) {
        hipLaunchKernelGGL((gm_gen32_kernel<G, DT>), dim3(blocks), dim3(256), 0, st, states + first,
                           states + first, m, n, (char*)out + first * n * es);
        return hipGetLastError();
      });
    }
  }
  while (seclen > unit && (uint64_t)count * ((n + seclen - 1) / seclen) < 1024 * Q) seclen /= 2;
  if ((uint64_t)count >= kFillWaves * Q || n < 2 * seclen || n < 3 * unit) {
    return launch_ranges(count, 256, 4 * Q, [&](uint64_t first, uint32_t m, uint32_t blocks) {
      hipLaunchKernelGGL((gmx_kernel<G, DT, false>), dim3(blocks), dim3(256), 0, st, states + first, states + first, m,
                         n, 1u, n, (char*)out + first * n * es, T.gmx, T.gm);
      return hipGetLastError();
    });
  }
  // (at most 2 kFillWaves wavefronts from here on)
  while ((uint64_t)count * ((n + 2 * seclen - 1) / (2 * seclen)) >= kFillWaves * Q) seclen *= 2;
  const uint32_t nsec = (uint32_t)((n + seclen - 1) / seclen);
  const uint32_t blocks = (uint32_t)((((uint64_t)count * nsec + Q - 1) / Q + 3) / 4);
  hipLaunchKernelGGL((gmx_kernel<G, DT, true>), dim3(blocks), dim3(256), 0, st, states, nullptr, count, n, nsec, seclen,
                     (char*)out, T.gmx, T.gm);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  JumpSpec js;
  js.fixed = n;
  return launch_jump_g<G>(T, states, count, js, nullptr, st);
}

// One stream: sections from one advance of the states on, so that a short
// call's time is that of a few; eight or more once they fill the chip's SIMDs.
// (10^5 outputs by copies, jumps and sections of 4096 in launches of their own,
// and so: GM61 232 and 21 us, GQ58.3 138 and 24; 10^7: 305 and 148, 190 and 91.)
template <int G>
uint64_t single_seclen(uint64_t n) {
  constexpr uint64_t Q = Mx<G>::Q;
  constexpr uint64_t unit = G == 6 ? kGmxSteps / 8 * 9 : kGmxSteps;
  uint64_t seclen = unit;
  while (seclen < 8 * unit && (n + seclen - 1) / seclen > 1024 * Q) seclen *= 2;
  while ((n + 2 * seclen - 1) / (2 * seclen) >= kFillWaves * Q) seclen *= 2;
  return seclen;
}

template <int G>
hipError_t launch_single_g(const DeviceTables& T, int dtype, const GmState* base, GmState* sout, uint64_t n, void* out,
                           hipStream_t st) {
  constexpr uint64_t Q = Mx<G>::Q;
  const uint64_t seclen = single_seclen<G>(n);
  const uint32_t nsec = (uint32_t)((n + seclen - 1) / seclen);
  const dim3 grid((uint32_t)((nsec + 4 * Q - 1) / (4 * Q))), block(256);
  switch (dtype) {
    case PRAND_U32:
      hipLaunchKernelGGL((gmx_kernel<G, PRAND_U32, true>), grid, block, 0, st, base, sout, 1u, n, nsec, seclen,
                         (char*)out, T.gmx, T.gm);
      break;
    case PRAND_F32:
      hipLaunchKernelGGL((gmx_kernel<G, PRAND_F32, true>), grid, block, 0, st, base, sout, 1u, n, nsec, seclen,
                         (char*)out, T.gmx, T.gm);
      break;
    default:
      hipLaunchKernelGGL((gmx_kernel<G, PRAND_F64, true>), grid, block, 0, st, base, sout, 1u, n, nsec, seclen,
                         (char*)out, T.gmx, T.gm);
      break;
  }
  return hipGetLastError();
}

template <int G>
hipError_t launch_gen_g(const DeviceTables& T, int dtype, GmState* states, uint32_t count, uint64_t n, void* out,
                        hipStream_t st) {
  switch (dtype) {
    case PRAND_U32: return launch_gen<G, PRAND_U32>(T, states, count, n, out, st);
    case PRAND_F32: return launch_gen<G, PRAND_F32>(T, states, count, n, out, st);
    default: return launch_gen<G, PRAND_F64>(T, states, count, n, out, st);
  }
}

}  // namespace

hipError_t launch_gm_generate(const DeviceTables& T, int gen, GmState* states, uint32_t count, uint64_t n, int dtype,
                              void* out, hipStream_t st) {
  switch (gen - PRAND_GM19) {
    case 0: return launch_gen_g<0>(T, dtype, states, count, n, out, st);
    case 1: return launch_gen_g<1>(T, dtype, states, count, n, out, st);
    case 2: return launch_gen_g<2>(T, dtype, states, count, n, out, st);
    case 3: return launch_gen_g<3>(T, dtype, states, count, n, out, st);
    case 4: return launch_gen_g<4>(T, dtype, states, count, n, out, st);
    case 5: return launch_gen_g<5>(T, dtype, states, count, n, out, st);
    case 6: return launch_gen_g<6>(T, dtype, states, count, n, out, st);
    default: return launch_gen_g<7>(T, dtype, states, count, n, out, st);
  }
}

hipError_t launch_gm_single(const DeviceTables& T, int gen, const GmState* base, GmState* sout, uint64_t n, int dtype,
                            void* out, hipStream_t st) {
  switch (gen - PRAND_GM19) {
    case 0: return launch_single_g<0>(T, dtype, base, sout, n, out, st);
    case 1: return launch_single_g<1>(T, dtype, base, sout, n, out, st);
    case 2: return launch_single_g<2>(T, dtype, base, sout, n, out, st);
    case 3: return launch_single_g<3>(T, dtype, base, sout, n, out, st);
    case 4: return launch_single_g<4>(T, dtype, base, sout, n, out, st);
    case 5: return launch_single_g<5>(T, dtype, base, sout, n, out, st);
    case 6: return launch_single_g<6>(T, dtype, base, sout, n, out, st);
    default: return launch_single_g<7>(T, dtype, base, sout, n, out, st);
  }
}

uint64_t gm_single_wavefronts(int gen, uint64_t n) {
  switch (gen - PRAND_GM19) {
    case 0: return (n / single_seclen<0>(n)) / Mx<0>::Q + 1;
    case 1: return (n / single_seclen<1>(n)) / Mx<1>::Q + 1;
    case 2: return (n / single_seclen<2>(n)) / Mx<2>::Q + 1;
    case 3: return (n / single_seclen<3>(n)) / Mx<3>::Q + 1;
    case 4: return (n / single_seclen<4>(n)) / Mx<4>::Q + 1;
    case 5: return (n / single_seclen<5>(n)) / Mx<5>::Q + 1;
    case 6: return (n / single_seclen<6>(n)) / Mx<6>::Q + 1;
    default: return (n / single_seclen<7>(n)) / Mx<7>::Q + 1;
  }
}

hipError_t launch_gm_jump(const DeviceTables& T, int gen, GmState* states, uint32_t count, const JumpSpec& js,
                          const GmState* base, hipStream_t st) {
  switch (gen - PRAND_GM19) {
    case 0: return launch_jump_g<0>(T, states, count, js, base, st);
    case 1: return launch_jump_g<1>(T, states, count, js, base, st);
    case 2: return launch_jump_g<2>(T, states, count, js, base, st);
    case 3: return launch_jump_g<3>(T, states, count, js, base, st);
    case 4: return launch_jump_g<4>(T, states, count, js, base, st);
    case 5: return launch_jump_g<5>(T, states, count, js, base, st);
    case 6: return launch_jump_g<6>(T, states, count, js, base, st);
    default: return launch_jump_g<7>(T, states, count, js, base, st);
  }
}

}  // namespace prand
