// Batched launch: task and tile records shared by the host planner
// (batch.hip) and the batch kernels (k_batch.hip).
#pragma once

#include <vector>

#include "prand_impl.h"

namespace prand {

// one task: the public prand_task, field for field
struct BatchTask {
  int32_t gen;
  int32_t dtype;
  uint64_t n;
  const void* state_in;
  void* state_out;
  void* out;
};
static_assert(sizeof(BatchTask) == sizeof(prand_task), "prand_task layout");

constexpr uint32_t kTileGen = 0;    // generate sections first .. first + nsec - 1
constexpr uint32_t kTileCopy = 1;   // n = 0: copy state_in to state_out
// section `first` of a long MT19937 task (kMtSection outputs each: whole
// 624-word blocks), started from the state the section-start kernel leaves
// in the scratch
constexpr uint32_t kTileMtSection = 2;
constexpr uint64_t kMtSection = 624ull << kMtBlkFirst;

// the work of one wavefront (an MT19937 tile's: of one workgroup)
struct BatchTile {
  uint32_t task;
  uint32_t kind;
  uint64_t first;      // first section of the tile
  uint64_t seclen;     // outputs per section (the task's last section may be shorter)
  uint32_t nsec;       // live sections in the tile
  uint32_t pad;
  uint64_t words;      // copy tiles: 32-bit words of the state
  uint64_t starts;     // byte offset of the tile's section start states in
                       // the batch scratch (MRG32K3A/LFSR113 and GM/GQ tiles)
};

// tiles are stored family by family: [reg | gm | mt | copy | cut]
// (MRG32K3A/LFSR113; GM/GQ; MT19937; n = 0; the further sections of MT19937
// tasks that are cut because the rest of the batch is shorter than they are,
// each of them one tile to the caller)
struct BatchCounts {
  uint32_t reg = 0, gm = 0, mt = 0, copy = 0, cut = 0;
  uint32_t mtsec = 0;   // MT19937 section tiles among the mt and cut ones
  uint32_t with_starts() const { return reg + gm; }
  uint32_t total() const { return with_starts() + mt + copy; }
};
constexpr int kFamReg = 0, kFamGm = 1, kFamMt = 2, kFamCopy = 3, kFamCut = 4, kBatchFamilies = 5;

// tile lists of a launch: MT19937 and copies, MRG32K3A/LFSR113, GM/GQ
constexpr int kListMt = 0, kListReg = 1, kListGm = 2, kBatchLists = 3;

struct BatchPlan {
  std::vector<BatchTile> tiles;
  BatchCounts n;
  uint64_t scratch_bytes = 0;
  // tile indices of the launch's lists, longest (estimated time) first,
  // indexed by kList*, and the whole-chip time of each
  std::vector<uint32_t> order[kBatchLists];
  double cost[kBatchLists] = {0, 0, 0};
};

// zero fields of a configuration replaced by the defaults
void batch_fill_defaults(prand_batch_config& c);
// cut tasks into tiles, family by family, each family longest first
// (PRAND_OK or an error code); MT19937 tasks longer than mt_section_min
// outputs are cut into kMtSection-output sections, and (may_cut: the MT19937
// tables are at hand) shorter ones that would outlast the rest of the batch
int batch_plan(const prand_task* tasks, uint32_t ntasks, const prand_batch_config& cfg, BatchPlan& plan,
               uint64_t mt_section_min, bool may_cut);
// MT19937 tasks of a batched launch above this many outputs (about 6 ms of a
// workgroup) run as sections
constexpr uint64_t kMtBatchSectionMin = 1ull << 24;

// the kernels of a batch, `waves` wavefronts (tiles) per workgroup
hipError_t launch_batch_starts(const DeviceTables& T, const BatchTile* tiles, uint32_t ntiles, const BatchTask* tasks,
                               char* scratch, uint32_t waves, hipStream_t st);
hipError_t launch_batch_reg(const BatchTile* tiles, uint32_t ntiles, const BatchTask* tasks, const char* scratch,
                            uint32_t waves, hipStream_t st);
hipError_t launch_batch_gm(const DeviceTables& T, const BatchTile* tiles, uint32_t ntiles, const BatchTask* tasks,
                           const char* scratch, uint32_t waves, hipStream_t st);
// MT19937 tiles and n = 0 copies
hipError_t launch_batch_mt(const BatchTile* tiles, uint32_t ntiles, const BatchTask* tasks, char* scratch,
                           hipStream_t st);
// start states of the MT19937 section tiles among tiles[0 .. ntiles): the
// task state moved first * kMtSection outputs on (one workgroup each)
hipError_t launch_batch_mt_starts(const DeviceTables& T, const BatchTile* tiles, uint32_t ntiles,
                                  const BatchTask* tasks, char* scratch, hipStream_t st);
// the reg kernel's tile counter, cleared by a small kernel (no memset node in a
// captured graph)
hipError_t launch_batch_reset(uint32_t* counter, hipStream_t st);
// workgroups of the persistent reg kernel resident on the chip at once (of
// `waves` wavefronts, LDS chunk width cw = 16 or 32)
uint32_t batch_reg_blocks(int cw, uint32_t waves, int num_cus);
// MT19937 and copy tiles, then GM/GQ tiles
hipError_t launch_batch_main(const DeviceTables& T, const BatchTile* tiles, const uint32_t* mt_order, uint32_t nmt,
                             const uint32_t* gm_order, uint32_t ngm, const BatchTask* tasks, char* scratch,
                             hipStream_t st);
hipError_t launch_batch_reg_persistent(int cw, const BatchTile* tiles, const uint32_t* order, uint32_t n,
                                       const BatchTask* tasks, char* scratch, uint32_t* counter, uint32_t waves,
                                       uint32_t blocks, hipStream_t st);
// all of them on one stream: section starts, MT19937, GM/GQ, MRG32K3A/LFSR113
hipError_t launch_batch_serial(const DeviceTables& T, const BatchTile* tiles, const BatchCounts& n,
                               const BatchTask* tasks, char* scratch, uint32_t waves, hipStream_t st);

}  // namespace prand
