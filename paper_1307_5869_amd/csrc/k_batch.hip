// Batched generation: many tasks (generator, state, length, dtype, output) of
// uneven sizes in one launch.
//
// The host cuts every task into tiles, one tile being the work of one
// wavefront: 64 lane-sections of a MRG32K3A / LFSR113 task, the GM/GQ sections
// that one 32-row operand of the matrix instructions holds (one of a v = 1
// ensemble, four of GM55 / GQ58.4, two of GQ58.3; dev_gmx.h); or the work of a
// workgroup: a whole MT19937 task or a section of a long one.  Sections are
// independent: each starts from the task's state jumped to its first output.
//
// A batched launch (prand_batch_launch) is a chain of kernels on one stream:
//  - batch_starts_kernel jumps every MRG32K3A/LFSR113/GM/GQ section to its
//    start and writes the state to the batch's scratch area (the jump code
//    needs many registers, so it runs apart from the generation loops);
//    sections of long MT19937 tasks (batch.hip) get theirs from
//    mt_section_start_kernel (k_mt19937.hip);
//  - batch_main_kernel runs MT19937 tasks and sections (and n = 0 copies), a
//    workgroup each, and the GM/GQ tiles, a wavefront each, in the order of
//    their lists, longest first (estimated time, by the host), so the long
//    tiles start at once and the short ones fill the end;
//  - batch_reg_persistent_kernel runs MRG32K3A/LFSR113 (its LDS sized by the
//    chunk width of the staging, the footprint the autotuner chooses): as many
//    workgroups as the chip holds at once, or fewer, which take the next tile of
//    their list from a device counter (cleared by batch_reset_kernel) until it is
//    used up.
// A counter costs 15 ns a tile: main by one took 10.5 ms for 2000 tasks of
// 10^3 .. 10^6 outputs in GM/GQ tiles of 256, 2.4 so; 10^7 GM19 numbers of one
// task 203 us and 67; 2000 MT19937 tasks of 100 .. 1000 96 and 23 (2000 tasks of
// 10^3 .. 10^7: 7.0 ms either way).
// Each tile runs the same routines as the one-generator kernels; the GM/GQ ones
// with the element type as a value, so that the kernel holds each generator's
// code once.  2000 tasks of 10^3 .. 10^7 outputs of all generators: 20.9 ms with
// a ballot or a lane per section for GM/GQ and a wavefront per MT19937 task, 7.0
// so.
//
// The serving loop keeps one grid kernel per family (batch_reg_kernel,
// batch_gmx_kernel, batch_mt_kernel) on its iteration stream: its iterations
// are small, and their length is set by the longest chunk.
#include <algorithm>

#include "dev_gm.h"
#include "dev_gmx.h"
#include "dev_lfsr.h"
#include "dev_mrg.h"
#include "dev_mt.h"
#include "prand_batch.h"
#include "regstream.h"

namespace prand {
namespace {

constexpr int kBatchCW = 32;   // MRG32K3A/LFSR113 staging chunk of the grid kernels

// section geometry of a MRG32K3A/LFSR113 tile: lane l takes section first + l
struct Sect {
  bool live;
  uint64_t start, len;
  bool last;
};
__device__ __forceinline__ Sect section_of(const BatchTile& tl, const BatchTask& tk) {
  const int gi = threadIdx.x & 63;
  Sect s;
  s.live = (uint32_t)gi < tl.nsec;
  s.start = (tl.first + (uint64_t)gi) * tl.seclen;
  s.len = s.live ? (s.start + tl.seclen <= tk.n ? tl.seclen : tk.n - s.start) : 0;
  s.last = s.live && s.start + s.len == tk.n;
  return s;
}

// the tile index of this wavefront, known to the compiler as uniform across
// it, so the tile and task fields it loads live in scalar registers
__device__ __forceinline__ uint32_t wave_index() {
  return __builtin_amdgcn_readfirstlane(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6));
}

// ---------------------------------------------------------------- starts
template <class G>
__device__ __noinline__ void start_reg(const BatchTile& tl, const BatchTask& tk, char* scratch,
                                       const uint32_t* ladder) {
  const Sect s = section_of(tl, tk);
  if (!s.live) return;
  typename G::State st = *(const typename G::State*)tk.state_in;
  if (s.start) G::jump(st, s.start, ladder);
  ((typename G::State*)(scratch + tl.starts))[threadIdx.x & 63] = st;
}

// lane e of a section's group: element e
template <int G>
__device__ __noinline__ void start_gm(const BatchTile& tl, const BatchTask& tk, char* scratch,
                                      const uint64_t* ladder) {
  constexpr int per = 32 / gm::Mx<G>::Q;   // lanes per section
  const int lane = threadIdx.x & 63, q = lane / per, e = lane % per;
  if ((uint32_t)q >= tl.nsec || q >= gm::Mx<G>::Q || e >= gm::Mx<G>::S) return;
  uint64_t xc, xp;
  const uint32_t off = gm::load_at<G>((const GmState*)tk.state_in, e, (tl.first + q) * tl.seclen, xc, xp, ladder);
  GmState* dst = (GmState*)(scratch + tl.starts) + q;
  dst->xc[e] = xc;
  dst->xp[e] = xp;
  if (e == 0) {
    dst->off = off;
    dst->pad = 0;
  }
}

__global__ void __launch_bounds__(256) batch_starts_kernel(const BatchTile* __restrict__ tiles, uint32_t ntiles,
                                                           const BatchTask* __restrict__ tasks, char* scratch,
                                                           DeviceTables T) {
  const uint32_t t = wave_index();
  if (t >= ntiles) return;
  const BatchTile tl = tiles[t];
  const BatchTask tk = tasks[tl.task];
  switch (tk.gen) {
    case PRAND_MRG32K3A: start_reg<mrg::MrgGen>(tl, tk, scratch, T.mrg); break;
    case PRAND_LFSR113: start_reg<lfsr::LfsrGen>(tl, tk, scratch, T.lfsr); break;
    case PRAND_GM19: start_gm<0>(tl, tk, scratch, T.gm); break;
    case PRAND_GM29: start_gm<1>(tl, tk, scratch, T.gm); break;
    case PRAND_GM31: start_gm<2>(tl, tk, scratch, T.gm); break;
    case PRAND_GM55: start_gm<3>(tl, tk, scratch, T.gm); break;
    case PRAND_GM61: start_gm<4>(tl, tk, scratch, T.gm); break;
    case PRAND_GQ58X1: start_gm<5>(tl, tk, scratch, T.gm); break;
    case PRAND_GQ58X3: start_gm<6>(tl, tk, scratch, T.gm); break;
    case PRAND_GQ58X4: start_gm<7>(tl, tk, scratch, T.gm); break;
    default: break;
  }
}

// ------------------------------------------------------- MRG32K3A/LFSR113
template <class G, int DT, int CW = kBatchCW>
__device__ __forceinline__ void gen_reg(const BatchTile& tl, const BatchTask& tk, uint32_t* lds,
                                        const char* scratch) {
  constexpr int es = (DT == PRAND_F64) ? 8 : 4;
  const Sect s = section_of(tl, tk);
  void* o = (char*)tk.out + (s.live ? s.start : 0) * es;
  const typename G::State* in = (const typename G::State*)(scratch + tl.starts) + (threadIdx.x & 63);
  regstream_wave<G, DT, CW, false>(lds, s.live, in, 0, s.len, o,
                                         s.last ? (typename G::State*)tk.state_out : nullptr, nullptr);
}

__global__ void __launch_bounds__(256) batch_reg_kernel(const BatchTile* __restrict__ tiles, uint32_t ntiles,
                                                        const BatchTask* __restrict__ tasks, const char* scratch) {
  __shared__ __align__(16) uint32_t lds[4][RegStage<kBatchCW>::kWaveWords];
  const uint32_t t = wave_index();
  if (t >= ntiles) return;
  uint32_t* mine = lds[(threadIdx.x >> 6) & 3];
  const BatchTile tl = tiles[t];
  const BatchTask tk = tasks[tl.task];
  const bool mrg = tk.gen == PRAND_MRG32K3A;
  switch (tk.dtype) {
    case PRAND_U32:
      if (mrg) gen_reg<mrg::MrgGen, PRAND_U32>(tl, tk, mine, scratch);
      else gen_reg<lfsr::LfsrGen, PRAND_U32>(tl, tk, mine, scratch);
      break;
    case PRAND_F32:
      if (mrg) gen_reg<mrg::MrgGen, PRAND_F32>(tl, tk, mine, scratch);
      else gen_reg<lfsr::LfsrGen, PRAND_F32>(tl, tk, mine, scratch);
      break;
    default:
      if (mrg) gen_reg<mrg::MrgGen, PRAND_F64>(tl, tk, mine, scratch);
      else gen_reg<lfsr::LfsrGen, PRAND_F64>(tl, tk, mine, scratch);
      break;
  }
}

// ------------------------------------------------------------------ GM/GQ
template <int G>
__device__ __forceinline__ void gen_gm(const BatchTile* tile, const BatchTask* tasks, const char* scratch,
                                    const GmxTable* tables, uint32_t* lds) {
  const BatchTask& tk = tasks[tile->task];
  const uint64_t first = gm::gmx_uniform(tile->first * tile->seclen), seclen = gm::gmx_uniform(tile->seclen), n = gm::gmx_uniform(tk.n);
  const uint64_t out = gm::gmx_uniform((uint64_t)tk.out), sout = gm::gmx_uniform((uint64_t)tk.state_out);
  const uint64_t starts = gm::gmx_uniform((uint64_t)(scratch + tile->starts)), table = gm::gmx_uniform((uint64_t)(tables + G));
  const uint32_t nsec = __builtin_amdgcn_readfirstlane(tile->nsec);
  const int dtype = __builtin_amdgcn_readfirstlane(tk.dtype);
  const uint64_t es = dtype == PRAND_F64 ? 8 : 4;
  auto sec = [&](int q) {
    gm::GmxSec r{nullptr, 0, 0, nullptr, nullptr};
    if ((uint32_t)q < nsec) {
      const uint64_t start = first + q * seclen;
      r.in = (const GmState*)starts + q;
      r.n = start + seclen <= n ? seclen : n - start;
      r.out = (char*)out + start * es;
      r.sout = start + r.n == n ? (GmState*)sout : nullptr;
    }
    return r;
  };
  gm::gmx_wave<G, gm::kAnyType, false>(sec, (const GmxTable*)table, nullptr, lds, dtype);
}

__device__ __forceinline__ void gm_tile(const BatchTile* tile, const BatchTask* tasks, const char* scratch,
                                        const GmxTable* table, uint32_t* lds) {
  switch (tasks[tile->task].gen) {
    case PRAND_GM19: gen_gm<0>(tile, tasks, scratch, table, lds); break;
    case PRAND_GM29: gen_gm<1>(tile, tasks, scratch, table, lds); break;
    case PRAND_GM31: gen_gm<2>(tile, tasks, scratch, table, lds); break;
    case PRAND_GM55: gen_gm<3>(tile, tasks, scratch, table, lds); break;
    case PRAND_GM61: gen_gm<4>(tile, tasks, scratch, table, lds); break;
    case PRAND_GQ58X1: gen_gm<5>(tile, tasks, scratch, table, lds); break;
    case PRAND_GQ58X3: gen_gm<6>(tile, tasks, scratch, table, lds); break;
    default: gen_gm<7>(tile, tasks, scratch, table, lds); break;
  }
}

__global__ void __launch_bounds__(256, 4) batch_gmx_kernel(const BatchTile* __restrict__ tiles, uint32_t ntiles,
                                                        const BatchTask* __restrict__ tasks, const char* scratch,
                                                        const GmxTable* __restrict__ table) {
  __shared__ uint32_t lds[4][gm::kGmxLds];
  const uint32_t t = wave_index();
  if (t >= ntiles) return;
  gm_tile(tiles + t, tasks, scratch, table, lds[(threadIdx.x >> 6) & 3]);
}

// --------------------------------------------------- MT19937 and n = 0 tasks
// A whole MT19937 task, or one kMtSection-output section of a long one, by a
// workgroup of mt::kGroup threads: the section starts from its state in the
// scratch; a section that is not the task's last leaves its end state in that
// same slot (read by this workgroup only, before it is written).
__device__ __forceinline__ void mt_tile(const BatchTile& tl, const BatchTask& tk, char* scratch, uint32_t* ring) {
  if (tl.kind == kTileCopy) {
    // n = 0: the output state is the input state
    const uint32_t* a = (const uint32_t*)tk.state_in;
    uint32_t* b = (uint32_t*)tk.state_out;
    for (uint32_t i = threadIdx.x; i < tl.words; i += mt::kGroup) b[i] = a[i];
    return;
  }
  const MtState* in = (const MtState*)tk.state_in;
  MtState* out = (MtState*)tk.state_out;
  uint64_t n = tk.n, start = 0;
  if (tl.kind == kTileMtSection) {
    MtState* slot = (MtState*)(scratch + tl.starts);
    start = tl.first * tl.seclen;
    n = (tk.n - start < tl.seclen) ? tk.n - start : tl.seclen;
    in = slot;
    if (start + n < tk.n) out = slot;
  }
  switch (tk.dtype) {
    case PRAND_U32: mt::gen_group<PRAND_U32>(ring, in, out, n, (char*)tk.out + start * 4); break;
    case PRAND_F32: mt::gen_group<PRAND_F32>(ring, in, out, n, (char*)tk.out + start * 4); break;
    default: mt::gen_group<PRAND_F64>(ring, in, out, n, (char*)tk.out + start * 8); break;
  }
}

__global__ void __launch_bounds__(mt::kGroup) batch_mt_kernel(const BatchTile* __restrict__ tiles,
                                                              const BatchTask* __restrict__ tasks, char* scratch) {
  __shared__ uint32_t ring[mt::kRing];
  const BatchTile tl = tiles[blockIdx.x];
  mt_tile(tl, tasks[tl.task], scratch, ring);
}

// ---------------------------------------------------------- persistent
__global__ void batch_reset_kernel(uint32_t* counter) { *counter = 0; }

// the next entry of a tile list for this wavefront (uniform across it)
__device__ __forceinline__ uint32_t next_tile(uint32_t* counter) {
  uint32_t k = 0;
  if ((threadIdx.x & 63) == 0) k = atomicAdd(counter, 1u);
  return __builtin_amdgcn_readfirstlane(__shfl(k, 0));
}

template <int CW>
struct RegLds {
  static constexpr int kWords = RegStage<CW>::kWaveWords;
};

// MRG32K3A/LFSR113 tiles, LDS staging chunks of CW words
template <int CW>
__global__ void __launch_bounds__(256) batch_reg_persistent_kernel(const BatchTile* __restrict__ tiles,
                                                                   const uint32_t* __restrict__ order, uint32_t n,
                                                                   const BatchTask* __restrict__ tasks,
                                                                   char* scratch, uint32_t* counter) {
  __shared__ __align__(16) uint32_t lds[4][RegLds<CW>::kWords];
  uint32_t* mine = lds[(threadIdx.x >> 6) & 3];
  for (;;) {
    const uint32_t k = next_tile(counter);
    if (k >= n) break;
    const BatchTile tl = tiles[order[k]];
    const BatchTask tk = tasks[tl.task];
    const bool mrg = tk.gen == PRAND_MRG32K3A;
    switch (tk.dtype) {
      case PRAND_U32:
        if (mrg) gen_reg<mrg::MrgGen, PRAND_U32, CW>(tl, tk, mine, scratch);
        else gen_reg<lfsr::LfsrGen, PRAND_U32, CW>(tl, tk, mine, scratch);
        break;
      case PRAND_F32:
        if (mrg) gen_reg<mrg::MrgGen, PRAND_F32, CW>(tl, tk, mine, scratch);
        else gen_reg<lfsr::LfsrGen, PRAND_F32, CW>(tl, tk, mine, scratch);
        break;
      default:
        if (mrg) gen_reg<mrg::MrgGen, PRAND_F64, CW>(tl, tk, mine, scratch);
        else gen_reg<lfsr::LfsrGen, PRAND_F64, CW>(tl, tk, mine, scratch);
        break;
    }
    wave_lds_sync();
  }
}

// MT19937 tasks and sections (and n = 0 copies), a workgroup each, then GM/GQ
// tiles, a wavefront each.  The MT19937 ones, whose chains are the longest of the
// batch, are dispatched first, and issue before the GM/GQ wavefronts they share a
// SIMD with: they are few, and wait for one another at every turn.  first: the
// launch's first workgroup of the batch's.
__global__ void __launch_bounds__(mt::kGroup, 4)
    batch_main_kernel(const BatchTile* __restrict__ tiles, const uint32_t* __restrict__ mt_order, uint32_t nmt,
                      const uint32_t* __restrict__ gm_order, uint32_t ngm, const BatchTask* __restrict__ tasks,
                      char* scratch, uint32_t first, const GmxTable* __restrict__ table) {
  __shared__ uint32_t ring[mt::kRing];
  __shared__ uint32_t lds[4][gm::kGmxLds];
  const uint32_t b = first + blockIdx.x;
  if (b < nmt) {
    __builtin_amdgcn_s_setprio(3);
    const BatchTile tl = tiles[mt_order[b]];
    mt_tile(tl, tasks[tl.task], scratch, ring);
    return;
  }
  const uint64_t k = (uint64_t)(b - nmt) * (mt::kGroup / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (k < ngm) gm_tile(tiles + gm_order[k], tasks, scratch, table, lds[threadIdx.x >> 6]);
}

uint32_t blocks_for(uint32_t ntiles, uint32_t waves) { return (ntiles + waves - 1) / waves; }

// resident workgroups of `waves` wavefronts on the whole chip
template <class K>
uint32_t resident_blocks(K kernel, uint32_t waves, int num_cus) {
  int per_cu = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, (int)(64 * waves), 0) != hipSuccess ||
      per_cu < 1)
    per_cu = 1;
  return (uint32_t)per_cu * (uint32_t)(num_cus > 0 ? num_cus : 1);
}

}  // namespace

hipError_t launch_batch_reset(uint32_t* counter, hipStream_t st) {
  hipLaunchKernelGGL(batch_reset_kernel, dim3(1), dim3(1), 0, st, counter);
  return hipGetLastError();
}

uint32_t batch_reg_blocks(int cw, uint32_t waves, int num_cus) {
  return cw == 16 ? resident_blocks(batch_reg_persistent_kernel<16>, waves, num_cus)
                  : resident_blocks(batch_reg_persistent_kernel<32>, waves, num_cus);
}

hipError_t launch_batch_main(const DeviceTables& T, const BatchTile* tiles, const uint32_t* mt_order, uint32_t nmt,
                             const uint32_t* gm_order, uint32_t ngm, const BatchTask* tasks, char* scratch,
                             hipStream_t st) {
  return launch_ranges((uint64_t)nmt + blocks_for(ngm, mt::kGroup / 64), mt::kGroup, 1,
                       [&](uint64_t first, uint32_t, uint32_t blocks) {
                         hipLaunchKernelGGL(batch_main_kernel, dim3(blocks), dim3(mt::kGroup), 0, st, tiles, mt_order,
                                            nmt, gm_order, ngm, tasks, scratch, (uint32_t)first, T.gmx);
                         return hipGetLastError();
                       });
}

hipError_t launch_batch_reg_persistent(int cw, const BatchTile* tiles, const uint32_t* order, uint32_t n,
                                       const BatchTask* tasks, char* scratch, uint32_t* counter, uint32_t waves,
                                       uint32_t blocks, hipStream_t st) {
  if (!n) return hipSuccess;
  blocks = std::min<uint32_t>(blocks, blocks_for(n, waves));
  const dim3 grid(blocks), block(64 * waves);
  if (cw == 16)
    hipLaunchKernelGGL(batch_reg_persistent_kernel<16>, grid, block, 0, st, tiles, order, n, tasks, scratch,
                       counter);
  else
    hipLaunchKernelGGL(batch_reg_persistent_kernel<32>, grid, block, 0, st, tiles, order, n, tasks, scratch,
                       counter);
  return hipGetLastError();
}

hipError_t launch_batch_starts(const DeviceTables& T, const BatchTile* tiles, uint32_t ntiles, const BatchTask* tasks,
                               char* scratch, uint32_t waves, hipStream_t st) {
  return launch_ranges(ntiles, 64 * waves, waves, [&](uint64_t first, uint32_t m, uint32_t blocks) {
    hipLaunchKernelGGL(batch_starts_kernel, dim3(blocks), dim3(64 * waves), 0, st, tiles + first, m, tasks, scratch, T);
    return hipGetLastError();
  });
}

hipError_t launch_batch_reg(const BatchTile* tiles, uint32_t ntiles, const BatchTask* tasks, const char* scratch,
                            uint32_t waves, hipStream_t st) {
  return launch_ranges(ntiles, 64 * waves, waves, [&](uint64_t first, uint32_t m, uint32_t blocks) {
    hipLaunchKernelGGL(batch_reg_kernel, dim3(blocks), dim3(64 * waves), 0, st, tiles + first, m, tasks, scratch);
    return hipGetLastError();
  });
}

hipError_t launch_batch_gm(const DeviceTables& T, const BatchTile* tiles, uint32_t ntiles, const BatchTask* tasks,
                           const char* scratch, uint32_t waves, hipStream_t st) {
  return launch_ranges(ntiles, 64 * waves, waves, [&](uint64_t first, uint32_t m, uint32_t blocks) {
    hipLaunchKernelGGL(batch_gmx_kernel, dim3(blocks), dim3(64 * waves), 0, st, tiles + first, m, tasks, scratch, T.gmx);
    return hipGetLastError();
  });
}

hipError_t launch_batch_mt(const BatchTile* tiles, uint32_t ntiles, const BatchTask* tasks, char* scratch,
                           hipStream_t st) {
  return launch_ranges(ntiles, mt::kGroup, 1, [&](uint64_t first, uint32_t, uint32_t blocks) {
    hipLaunchKernelGGL(batch_mt_kernel, dim3(blocks), dim3(mt::kGroup), 0, st, tiles + first, tasks, scratch);
    return hipGetLastError();
  });
}

hipError_t launch_batch_serial(const DeviceTables& T, const BatchTile* tiles, const BatchCounts& n,
                               const BatchTask* tasks, char* scratch, uint32_t waves, hipStream_t st) {
  const BatchTile* gm = tiles + n.reg;
  const BatchTile* mt = tiles + n.with_starts();
  hipError_t e = launch_batch_starts(T, tiles, n.with_starts(), tasks, scratch, waves, st);
  if (e == hipSuccess && n.mtsec) e = launch_batch_mt_starts(T, mt, n.mt, tasks, scratch, st);
  if (e == hipSuccess) e = launch_batch_mt(mt, n.mt + n.copy, tasks, scratch, st);
  if (e == hipSuccess) e = launch_batch_gm(T, gm, n.gm, tasks, scratch, waves, st);
  if (e == hipSuccess) e = launch_batch_reg(tiles, n.reg, tasks, scratch, waves, st);
  return e;
}

}  // namespace prand
