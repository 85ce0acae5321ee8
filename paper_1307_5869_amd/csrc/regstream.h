// Generation for generators whose whole state fits in a lane's registers
// (MRG32K3A, LFSR113): one lane per section of a stream.
//
// A section starts from a state jumped to its first output and fills a
// contiguous run of the output.  The 64 runs of a wavefront lie in 64
// different places, so each lane produces its outputs in chunks of CW words
// (CW = 32: 128 bytes, 32 u32/f32 or 16 f64 values), parks them in LDS, and
// the wavefront stores them transposed: in each store instruction the CW/4
// consecutive lanes of a group write the 16-byte pieces of one chunk (CW = 32:
// eight whole 128-byte lines per instruction).  A lane's chunks are the
// aligned 4 CW-byte blocks of memory that its run touches, whatever the run's
// address (any multiple of the element size): only its first and last chunk
// may be partial.  A round in which a lane's chunk is partial makes its words
// one by one, all lanes together (four at a time left out that no lane's run
// covers); the 16-byte pieces that the run covers are stored as the others are,
// the words of a piece it covers in part by the lane.
// (Runs that did not start on 16 bytes used to be stored word by word, lane by
// lane: 10007 LFSR113 streams of 4999 f32 took 252 us, now 70 us.)  A lane
// whose run is shorter sits out the later rounds.
//
// regstream_wave() is the wavefront routine shared by the many-stream kernel
// below and by the batched generation kernel.
#pragma once

#include <cstdlib>
#include <type_traits>

#include "prand_impl.h"

namespace prand {

template <int CW>
struct RegStage {
  static constexpr int kRowWords = CW + 4;            // padded row, 16-byte aligned
  static constexpr int kWaveWords = 64 * kRowWords;   // LDS words per wavefront
};

template <int DT>
__device__ __forceinline__ void put_word(void* out, uint64_t i, uint32_t w, double f64v) {
  if (DT == PRAND_U32) ((uint32_t*)out)[i] = w;
  else if (DT == PRAND_F32) ((float*)out)[i] = (float)(w >> 8) * 0x1p-24f;
  else ((double*)out)[i] = f64v;
}

// One lane's section: live lanes start from *in (jumped `start` outputs
// ahead: by the jump matrix sec_mat when it is given, else by the bytes of
// the distance), write `len` values at `out` (element pointer of the run) and, when
// `sout` is set, store the advanced state there.  All 64 lanes must call.
// kJump = false: the caller guarantees start == 0 (no jump code is built).
// unit: bytes that the chunks are aligned to (16: short runs, which then touch
// fewer of them; 0: the lanes store their words by themselves).  drop: outputs to leave out before the first.
//
// G: State, Regs, static load(State) -> Regs, static save(Regs) -> State,
// static jump(State&, uint64_t distance, const uint32_t* ladder),
// static apply(State&, const uint32_t* jump matrix),
// static next(Regs&) -> uint32_t word, static f64(uint32_t) -> double.
template <class G, int DT, int CW, bool kJump = true>
__device__ __forceinline__ void regstream_wave(uint32_t* rows, bool live, const typename G::State* in, uint64_t start,
                                               uint64_t len, void* out, typename G::State* sout,
                                               const uint32_t* __restrict__ ladder,
                                               const uint32_t* __restrict__ sec_mat = nullptr,
                                               uint32_t unit = 4 * CW, uint32_t drop = 0) {
  constexpr int kPieces = CW / 4;                            // 16-byte pieces per chunk
  constexpr int kw = (DT == PRAND_F64) ? 2 : 1;               // words per value
  constexpr int es = 4 * kw;
  const int lane = threadIdx.x & 63;
  typename G::State st = {};
  if (live) {
    st = *in;
    if (kJump && sec_mat) G::apply(st, sec_mat);
    else if (kJump && start) G::jump(st, start, ladder);
  }
  typename G::Regs r = G::load(st);
  for (uint32_t i = 0; i < drop; i++) (void)G::next(r);
  // the run's frame: its chunks, the first of which it enters `head` words
  // on and the last of which it fills up to `tail` words (1 .. CW)
  const bool framed = unit && __all(!live || (uintptr_t)out % es == 0);
  const uint32_t head = live ? (uint32_t)((uintptr_t)out & (unit - 1)) / 4 : 0;
  const uint64_t total = (live && framed) ? head + len * kw : 0;   // words from the frame's start
  const uint32_t mine = (uint32_t)((total + CW - 1) / CW);         // chunks (0: none)
  const uint32_t tail = mine ? (uint32_t)(total - (uint64_t)(mine - 1) * CW) : 0;
  // chunks that any lane has; chunks below which every lane's are whole,
  // but for the first where a lane has a head
  uint32_t rounds = mine, even = mine ? mine - (tail < CW) : ~0u;
  const uint32_t first = __builtin_amdgcn_readfirstlane(mine);
  if (__all(mine == first && even == first)) {   // alike and whole in all lanes (40000 streams of 256 u32 19.0 -> 17.7 us)
    rounds = even = first;
  } else {
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t r1 = __shfl_xor(rounds, o), e1 = __shfl_xor(even, o);
      rounds = r1 > rounds ? r1 : rounds;
      even = e1 < even ? e1 : even;
    }
  }
  if (rounds) {
    const uint32_t skip = __any(head != 0) ? 1 : 0;   // chunks 0 .. skip - 1 may have a head
    // piece (lane % kPieces) of each source lane's chunk, one source lane per
    // store instruction: its address in chunk 0, and the chunks in which the
    // run covers it
    const int p4 = 4 * (lane % kPieces);
    char* const base = live ? (char*)out - 4 * (uint64_t)head : nullptr;
    char* dst[kPieces];
    uint32_t from[kPieces], whole[kPieces];   // from <= chunk < whole
#pragma unroll
    for (int i = 0; i < kPieces; i++) {
      const int src = i * (64 / kPieces) + lane / kPieces;
      dst[i] = (char*)__shfl((unsigned long long)base, src) + 4 * p4;
      const uint32_t chunks = __shfl(mine, src), ht = __shfl(head | tail << 8, src);
      from[i] = (int)(ht & 255) > p4 ? 1 : 0;
      whole[i] = chunks - (chunks && (int)(ht >> 8) < p4 + 4 ? 1 : 0);
    }
    uint32_t* row = rows + lane * RegStage<CW>::kRowWords;
    for (uint32_t rd = 0; rd < rounds; rd++) {
      // all: this chunk is whole for every live lane; parts: partial for one;
      // otherwise whole for the lanes that have it
      const bool all = rd >= skip && rd < even;
      const bool parts = !all && __any((rd == 0 && head) || (rd + 1 == mine && tail < CW));
      if (!parts) {
        if (rd < mine) {
#pragma unroll
          for (int q = 0; q < kPieces; q++) {
            uint4 v;
            if (DT == PRAND_F64) {
              const double a = G::f64(G::next(r)), b = G::f64(G::next(r));
              const uint64_t ua = __double_as_longlong(a), ub = __double_as_longlong(b);
              v = make_uint4((uint32_t)ua, (uint32_t)(ua >> 32), (uint32_t)ub, (uint32_t)(ub >> 32));
            } else if (DT == PRAND_F32) {
              const uint32_t a = G::next(r), b = G::next(r), c = G::next(r), d = G::next(r);
              v = make_uint4(__float_as_uint((float)(a >> 8) * 0x1p-24f), __float_as_uint((float)(b >> 8) * 0x1p-24f),
                             __float_as_uint((float)(c >> 8) * 0x1p-24f), __float_as_uint((float)(d >> 8) * 0x1p-24f));
            } else {
              const uint32_t a = G::next(r), b = G::next(r), c = G::next(r), d = G::next(r);
              v = make_uint4(a, b, c, d);
            }
            *(uint4*)(row + 4 * q) = v;
          }
        }
      } else {
        // word by word, the lanes together: the words of the run in this chunk;
        // those of a 16-byte piece that the run covers in part are stored here
        const uint32_t w0 = rd ? 0 : head, w1 = rd + 1 < mine ? CW : (rd + 1 == mine ? tail : 0);
        char* const at = base + (uint64_t)rd * (4 * CW);
#pragma unroll
        for (uint32_t w4 = 0; w4 < CW; w4 += 4) {
          if (!__any(w4 + 4 > w0 && w4 < w1)) continue;   // no lane's
#pragma unroll
          for (uint32_t w = w4; w < w4 + 4; w += kw)
            if (w >= w0 && w < w1) {
              const uint32_t v = G::next(r);
              put_word<DT>(row + w, 0, v, DT == PRAND_F64 ? G::f64(v) : 0.0);
            }
        }
        // of the pieces covered in part: up to 3 words at the run's front and end
        const uint32_t h4 = (w0 + 3) / 4 * 4 < w1 ? (w0 + 3) / 4 * 4 : w1, t4 = w1 / 4 * 4 > h4 ? w1 / 4 * 4 : h4;
        typedef typename std::conditional<DT == PRAND_F64, uint64_t, uint32_t>::type Value;
#pragma unroll
        for (uint32_t k = 0; k < 4 - kw; k += kw) {
          if (w0 + k < h4) *(Value*)(at + 4 * (w0 + k)) = *(const Value*)(row + w0 + k);
          if (t4 + k < w1) *(Value*)(at + 4 * (t4 + k)) = *(const Value*)(row + t4 + k);
        }
      }
      wave_lds_sync();
      const uint64_t adv = (uint64_t)rd * (4 * CW);
      if (all) {
#pragma unroll
        for (int i = 0; i < kPieces; i++) {
          const int src = i * (64 / kPieces) + lane / kPieces;
          const uint4 v = *(const uint4*)(rows + src * RegStage<CW>::kRowWords + p4);
          if (whole[i]) store_out16<DT, (CW >= 32)>(dst[i] + adv, v);   // (0: a dead lane's)
        }
      } else {
#pragma unroll
        for (int i = 0; i < kPieces; i++) {
          const int src = i * (64 / kPieces) + lane / kPieces;
          const uint4 v = *(const uint4*)(rows + src * RegStage<CW>::kRowWords + p4);
          if (rd >= from[i] && rd < whole[i]) store_out16<DT, (CW >= 32)>(dst[i] + adv, v);
        }
      }
      wave_lds_sync();
    }
  }
  if (live) {
    if (!framed)   // a very short run, or an address that is no multiple of the element size
      for (uint64_t i = 0; i < len; i++) {
        const uint32_t w = G::next(r);
        put_word<DT>(out, i, w, DT == PRAND_F64 ? G::f64(w) : 0.0);
      }
    if (sout) *sout = G::save(r);
  }
}

// Many streams: lane gid owns section gid & (nsec - 1) of stream
// gid >> nsec_log2; the sections of a stream cover
// [j * seclen, min((j + 1) * seclen, n)) and sit in one wavefront (nsec <= 64),
// so the state read of every section precedes the write-back of the last.
// With sectab (the section-start table of seclen), section j > 0 starts from
// row j - 1 of it, else from jumps by the byte tables.
//
// lines: sections begin on chunks of the output, for all but the first to be
// whole.  Where starts may lie anywhere (jumps by bytes) and the sections leave
// room for it, the first is shorter by as much as the stream's output begins
// inside a chunk; with starts by the table it is longer by the rest of that
// chunk, which the others drop.
template <class G, int DT, int CW>
__global__ void __launch_bounds__(256) regstream_kernel(typename G::State* states, uint32_t count, uint64_t n,
                                                        int nsec_log2, uint64_t seclen, bool lines, uint32_t unit,
                                                        void* __restrict__ out, const uint32_t* __restrict__ ladder,
                                                        const uint32_t* __restrict__ sectab) {
  __shared__ __align__(16) uint32_t stage[4][RegStage<CW>::kWaveWords];
  const uint64_t gid = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const uint64_t nsec = 1ull << nsec_log2;
  const uint64_t s = gid >> nsec_log2, j = gid & (nsec - 1);
  constexpr int es = (DT == PRAND_F64) ? 8 : 4;
  const uint64_t inside = lines ? ((uintptr_t)out + s * n * es) % (4 * CW) / es : 0;
  const bool any = !sectab && (seclen << nsec_log2) >= n + CW - 1;
  const uint64_t less = any ? inside : 0;
  const uint64_t more = sectab && inside ? 4 * CW / es - inside : 0;
  const uint64_t start = j ? j * seclen + more - less : 0, next = (j + 1) * seclen + more - less;
  const bool live = s < count && (!j || start < n);
  const bool last = live && next >= n;
  const uint64_t len = live ? (last ? n : next) - start : 0;
  void* o = (char*)out + (s * n + start) * es;
  const uint32_t* sec_mat = (sectab && j) ? sectab + (j - 1) * G::kSectionWords : nullptr;
  regstream_wave<G, DT, CW>(stage[threadIdx.x >> 6], live, states + (live ? s : 0), start, len, o,
                            last ? states + s : nullptr, ladder, sec_mat, unit, live && j ? (uint32_t)more : 0);
}

// One stream: lane j owns section j (seclen outputs, the last one the rest).
template <class G, int DT>
__global__ void __launch_bounds__(256) regstream_single_kernel(typename G::State base, typename G::State* sout,
                                                               uint64_t n, uint32_t nsec, uint64_t seclen,
                                                               void* __restrict__ out,
                                                               const uint32_t* __restrict__ table) {
  __shared__ __align__(16) uint32_t stage[4][RegStage<32>::kWaveWords];
  const uint32_t j = blockIdx.x * blockDim.x + threadIdx.x;
  const bool live = j < nsec;
  const uint64_t start = live ? j * seclen : 0;
  const uint64_t len = live ? (j + 1 < nsec ? seclen : n - start) : 0;
  constexpr int es = (DT == PRAND_F64) ? 8 : 4;
  regstream_wave<G, DT, 32>(stage[threadIdx.x >> 6], live, &base, start, len, (char*)out + start * es,
                            live && j + 1 == nsec ? sout : nullptr, table);
}

// Sections of 32 outputs up to kSingleLanes of them: a short call's time is the
// chain of one section (1000 MRG32K3A numbers: 51 us by way of copies, jumps
// and sections of 256 in launches of their own, 18 us as this one).  Then 64
// and so on, as the starts (one matrix per nonzero byte of the distance) would
// come to cost as much as the outputs, up to 2 KB of them: in longer ones the
// 64 runs of a wavefront lie further apart than the caches join (10^9 f64
// MRG32K3A: 1.47 ms in sections of 2 KB, 1.79 of 4 KB; 10^9 u32: 0.82 of 2 KB,
// 1.04 of 4 KB, 0.84 of 1 KB), until the lanes would be more than
// kSingleMaxLanes.
constexpr uint64_t kSingleLanes = 1u << 18, kSingleMaxLanes = 1u << 22;

template <class G>
hipError_t launch_regstream_single(const typename G::State* base, typename G::State* sout, uint64_t n, int dtype,
                                   void* out, const uint32_t* table, hipStream_t st) {
  uint64_t seclen = 32;
  auto lanes = [&]() { return (n + seclen - 1) / seclen; };
  const uint64_t full = dtype == PRAND_F64 ? 256 : 512;   // 2 KB
  while (seclen < full && lanes() > kSingleLanes) seclen *= 2;
  while (lanes() > kSingleMaxLanes) seclen *= 2;
  const uint32_t nsec = (uint32_t)((n + seclen - 1) / seclen);
  const dim3 grid((nsec + 255) / 256), block(256);
  switch (dtype) {
    case PRAND_U32:
      hipLaunchKernelGGL((regstream_single_kernel<G, PRAND_U32>), grid, block, 0, st, *base, sout, n, nsec, seclen, out,
                         table);
      break;
    case PRAND_F32:
      hipLaunchKernelGGL((regstream_single_kernel<G, PRAND_F32>), grid, block, 0, st, *base, sout, n, nsec, seclen, out,
                         table);
      break;
    default:
      hipLaunchKernelGGL((regstream_single_kernel<G, PRAND_F64>), grid, block, 0, st, *base, sout, n, nsec, seclen, out,
                         table);
      break;
  }
  return hipGetLastError();
}

// CW of the register-state kernels: 32 unless PRAND_REG_CHUNK_WORDS=16
inline int regstream_chunk_words() {
  static int cw = -1;
  if (cw < 0) {
    const char* e = getenv("PRAND_REG_CHUNK_WORDS");
    cw = (e && atoi(e) == 16) ? 16 : 32;
  }
  return cw;
}

template <class G, int CW>
hipError_t launch_regstream_cw(typename G::State* states, uint32_t count, uint64_t n, const RegPlan& plan, int dtype,
                               void* out, const uint32_t* ladder, hipStream_t st) {
  const uint32_t unit = plan.unit > 4 * CW ? 4 * CW : plan.unit;
  return launch_ranges(count, 256, 256u >> plan.nsec_log2, [&](uint64_t first, uint32_t m, uint32_t blocks) {
    auto launch = [&](auto* kernel, size_t es) {
      hipLaunchKernelGGL(kernel, dim3(blocks), dim3(256), 0, st, states + first, m, n, plan.nsec_log2, plan.seclen,
                         plan.lines, unit, (void*)((char*)out + first * n * es), ladder, plan.sectab);
      return hipGetLastError();
    };
    return dtype == PRAND_U32   ? launch(regstream_kernel<G, PRAND_U32, CW>, 4)
           : dtype == PRAND_F32 ? launch(regstream_kernel<G, PRAND_F32, CW>, 4)
                                : launch(regstream_kernel<G, PRAND_F64, CW>, 8);
  });
}

template <class G>
hipError_t launch_regstream(typename G::State* states, uint32_t count, uint64_t n, const RegPlan& plan, int dtype,
                            void* out, const uint32_t* ladder, hipStream_t st) {
  return regstream_chunk_words() == 16 ? launch_regstream_cw<G, 16>(states, count, n, plan, dtype, out, ladder, st)
                                       : launch_regstream_cw<G, 32>(states, count, n, plan, dtype, out, ladder, st);
}

}  // namespace prand
