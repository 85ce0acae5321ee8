// Internal declarations shared by the host side and the HIP kernels of the
// PRAND library for gfx950.  Nothing here is part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <mutex>
#include <utility>
#include <vector>

#include "prand.h"

namespace prand {

constexpr int kMaxLimbs = 8;        // distances up to 2^512
constexpr int kLadder = 512;        // jump tables hold M^(2^b) for b < 512
constexpr int kJumpRows = kLadder + 8 * 256;   // and M^(d 2^(8 j)) for j < 8, d < 256

// ---- state blobs (layout documented in prand.h) ----
struct MtState {
  uint32_t mt[624];
  uint32_t idx;
  uint32_t pad[3];
};
struct MrgState {
  uint32_t x[3];   // x_n, x_{n-1}, x_{n-2}
  uint32_t y[3];   // y_n, y_{n-1}, y_{n-2}
};
struct LfsrState {
  uint32_t z[4];
};
struct GmState {
  uint64_t xp[32];  // x^(n-1)
  uint64_t xc[32];  // x^(n)
  uint32_t off;     // GQ58.3: words of the current 8-step block already consumed
  uint32_t pad;
};
static_assert(sizeof(MtState) == 2512, "MT19937 state layout");
static_assert(sizeof(MrgState) == 24, "MRG32K3A state layout");
static_assert(sizeof(LfsrState) == 16, "LFSR113 state layout");
static_assert(sizeof(GmState) == 520, "GM state layout");

// ---- MRG32K3A constants: matrices A, B of the paper's MRG32K3A section ----
constexpr uint32_t kMrgM1 = 4294967087u;   // 2^32 - 209
constexpr uint32_t kMrgM2 = 4294944443u;   // 2^32 - 22853
constexpr uint32_t kMrgA12 = 1403580u;     // a
constexpr uint32_t kMrgA13n = 810728u;     // -b
constexpr uint32_t kMrgA21 = 527612u;      // c
constexpr uint32_t kMrgA23n = 1370589u;    // -d

// ---- GM/GQ parameters of the paper's Table 2 ----
// g = p * 2^t; s = ensemble size, v = digit bits per element.
struct GmParams {
  uint64_t k, q, p;
  int t, v, s;
  int n0;  // M^N = 0 mod 2^t for N >= n0 (composite moduli only)
};
constexpr GmParams kGmParams[8] = {
    /* GM19   */ {15, 28, 524287ull, 0, 1, 32, 0},
    /* GM29   */ {4, 2, 536870909ull, 0, 1, 32, 0},
    /* GM31   */ {11, 14, 2147483647ull, 0, 1, 32, 0},
    /* GM55   */ {256, 176, 2251799813685119ull, 4, 4, 8, 2},
    /* GM61   */ {24, 74, 2305843009213693951ull, 0, 1, 32, 0},
    /* GQ58.1 */ {8, 48, 536870909ull, 29, 1, 32, 16},
    /* GQ58.3 */ {8, 48, 536870909ull, 29, 3, 12, 16},
    /* GQ58.4 */ {8, 48, 536870909ull, 29, 4, 8, 16},
};

// ---- GM/GQ generation by matrix instructions (dev_gmx.h) ----
// p = 2^e - c; digits of `bits` bits per coefficient (their values cover p
// several times over), positions of a fraction and their width (14: in two
// parts of 7), whether the top one is doubled, offset of the result in units
// of the fraction's last bit
struct GmxShape {
  int e;
  uint64_t c;
  int bits, digits, positions, width, top, delta;
};
constexpr GmxShape kGmxShape[8] = {
    /* GM19   */ {19, 1, 5, 4, 2, 14, 1, 64},
    /* GM29   */ {29, 3, 8, 4, 4, 11, 0, 600},
    /* GM31   */ {31, 1, 4, 8, 4, 11, 0, 64},
    /* GM55   */ {51, 129, 8, 7, 6, 11, 1, 800},
    /* GM61   */ {61, 1, 8, 8, 7, 11, 0, 1000},
    /* GQ58.1 */ {29, 3, 8, 4, 4, 11, 0, 600},
    /* GQ58.3 */ {29, 3, 4, 8, 4, 11, 0, 64},
    /* GQ58.4 */ {29, 3, 4, 8, 4, 11, 0, 64},
};
constexpr int kGmxSteps = 256;   // steps per state advance
// Product h (0 .. 7) of a state value takes the digit with this many digits
// below it: two of 16 bits' distance share a word of the data, or the two parts
// of one (products 2 i and 2 i + 1, the digit times 1 and 128)
constexpr int gmx_below(int bits, int h) {
  return bits == 8 ? (h >> 1 & 1) + 4 * (h >> 2) + 2 * (h & 1) : bits == 4 ? (h >> 1) + 4 * (h & 1) : h >> 1;
}
// the digits' factor in the operands (their largest is 128 * 256, or 16 * 128 * 2)
constexpr int gmx_factor(int width, int h) { return width == 11 ? 256 : (h & 1 ? 256 : 2); }
struct alignas(16) GmxTable {
  uint64_t mat[(kGmxSteps + 1) * 4];   // M^j mod p, j = 0 .. kGmxSteps
  // matrix operands (f16, gmx_factor times the digits) for steps 32 g + 1 ..
  // 32 g + 32: 8 per lane at [(64 g + lane) * 8]
  uint16_t coef[(kGmxSteps / 32) * 64 * 8];
};

inline bool is_gm(int gen) { return gen >= PRAND_GM19 && gen <= PRAND_GQ58X4; }

// Byte tables for block splitting with each generator's default variant:
// the stream of id starts id 2^e steps on (e = kGmByteE[G], kLfsrByteE, the
// default block exponents), applied as one matrix per nonzero byte d_j of
// id (id = sum d_j 2^(8 j)): entry [j][d] is the jump by d 2^(e + 8 j), so a
// stream costs at most 8 matrix applications instead of one per set bit.
constexpr int kGmByteE[8] = {23, 27, 27, 34, 34, 27, 27, 27};
constexpr int kLfsrByteE = 34;

// ---- device-resident jump tables (built once per context) ----
struct DeviceTables {
  // distances: one matrix per nonzero byte (MRG32K3A: of all 512 bits;
  // LFSR113 and GM/GQ: of the low 64 bits, one per set bit above them)
  uint32_t* mrg = nullptr;    // [64][256][18]: A^(d 2^(8 j)) mod m1 (row major), B^(d 2^(8 j)) mod m2
  uint32_t* lfsr = nullptr;   // [kJumpRows][4][32]: columns of T_c^(2^b), b < kLadder, then T_c^(d 2^(8 j)), [8][256]
  uint64_t* gm = nullptr;     // [8][kJumpRows][4]: (a b; c d) = M^(2^b) mod p, then M^(d 2^(8 j)) mod p
  uint64_t* gmbyte = nullptr;   // [8][8][256][4]: M^(d 2^(kGmByteE[G] + 8 j)) mod p
  GmxTable* gmx = nullptr;      // [8]
  uint64_t* gmneg = nullptr;    // [8][4]: M^(-n0) mod p (composite moduli; identity otherwise)
  uint32_t* lfsrbyte = nullptr; // [8][256][4][32]: columns of T_c^(d 2^(kLfsrByteE + 8 j))
  uint32_t* mt = nullptr;     // [kLadder][624]: bits of x^(2^b) mod phi (19937 used)
  uint32_t* mtdiglo = nullptr;  // [3][65536][624]: x^(d 2^(kMtDigitE + 16k)) mod phi
  uint32_t* mtdig8hi = nullptr; // [2][256][624]: x^(d 2^(kMtDigitE + 48 + 8j)) mod phi
  void* mttop = nullptr;        // [65536] MtState: the default state jumped t 2^(kMtDigitE + 48)
  uint32_t* mtblk = nullptr;    // [kMtBlkDigits][16][624]: x^(d 624 2^(kMtBlkUnit + 4 k)) mod phi
  uint32_t* mtinv = nullptr;    // [624]: x^(-1) mod phi
  void* defaults = nullptr;   // default state of each generator, 11 x 2560 bytes
};
constexpr size_t kDefaultStride = 2560;
// exponent of the MT19937 digit tables: the block-splitting block 2^432
constexpr int kMtDigitE = 432;
// whole-block MT19937 jumps, in units of 624 2^kMtBlkUnit outputs by hexadecimal
// digits (calls and tasks of up to 2^40 outputs); sections of batched and
// served tasks have 624 2^kMtBlkFirst outputs
constexpr int kMtBlkUnit = 8, kMtBlkDigits = 6;
constexpr int kMtBlkFirst = 10;
constexpr int kMtBlkPolys = 4 * kMtBlkDigits - (kMtBlkFirst - kMtBlkUnit);   // bits of a section number

// Order a wavefront's LDS writes before its later LDS reads (and reads before
// later writes) when the LDS block is private to the wavefront: LDS
// instructions of one wavefront execute in order, so only the compiler must
// be kept from reordering.  No workgroup barrier: wavefronts of one workgroup
// may run different amounts of work (or leave early).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The lowest nonzero byte of w (w != 0), taken out of it: its position is
// returned, its value left in d.  Lanes whose distances have bytes in different
// places then go through their matrices together, one per nonzero byte.
__device__ __forceinline__ int take_byte(uint64_t& w, uint32_t& d) {
  const int j = __builtin_ctzll(w) >> 3;
  d = (uint32_t)(w >> (8 * j)) & 255u;
  w ^= (uint64_t)d << (8 * j);
  return j;
}

// 16-byte output store of the bulk generators.  u32/f32 outputs are marked
// non-temporal (the kernel that writes them never reads them back) when the
// caller's store instructions cover whole 128-byte lines (kLines); f64
// outputs and partial-line pieces stay plain.  Measured against plain stores, in alternation on one
// box: MT19937 u32 0.912 -> 0.861 ms per 2^30 words, LFSR113 u32 0.82 ->
// 0.81 ms, MRG32K3A within noise; in f64 non-temporal stores were slower
// (MRG32K3A and LFSR113 by 4 %, and MT19937, whose two stores per lane each
// cover half of every 32-byte piece, took twice as long).
template <int DT, bool kLines = true>
__device__ __forceinline__ void store_out16(void* p, uint4 v) {
  if (DT == PRAND_F64 || !kLines) {
    *(uint4*)p = v;
  } else {
    typedef unsigned int U4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(1))) U4 GU4;
    U4 w = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(w, (GU4*)p);
  }
}

// A dispatch holds fewer than 2^32 work-items.  Launches of more than one per
// stream (or tile) go out in ranges of streams that each fit: `per_block` of them
// to a workgroup of `block` threads; launch(first, m, blocks) -> hipError_t takes
// streams first .. first + m - 1.
template <class F>
hipError_t launch_ranges(uint64_t count, uint32_t block, uint32_t per_block, F&& launch) {
  const uint64_t most = (uint64_t)(0xFFFFFFFFu / block) * per_block;
  hipError_t e = hipSuccess;
  for (uint64_t first = 0; first < count && e == hipSuccess; first += most) {
    const uint64_t m = count - first < most ? count - first : most;
    e = launch(first, (uint32_t)m, (uint32_t)((m + per_block - 1) / per_block));
  }
  return e;
}

// ---- launchers (one per kernel family); all enqueue on `st` ----
// Distances: `dist` holds nlimbs limbs per stream when per_stream, else one
// shared distance.  `ids` + `block_e`: distance id * 2^block_e (GQ58.3: in
// ensemble steps).  Exactly one of (dist, ids) is used; GM/GQ with neither:
// every stream moves `fixed` outputs.
constexpr int kMtSections = 1, kMtUnits = 2;
struct JumpSpec {
  uint64_t fixed = 0;
  const uint64_t* dist = nullptr;
  int nlimbs = 0;
  int per_stream = 0;
  const uint64_t* ids = nullptr;
  int block_e = 0;
  // MT19937 block splitting from the default state: the states of the top
  // 16 bits of an id (DeviceTables::mttop), or null
  const void* mt_top = nullptr;
  // MT19937, per-stream one-limb distances.  kMtSections: counted in whole
  // sections of 624 2^kMtBlkFirst outputs (by the whole-block digits where the
  // state sits on a block boundary and the distance is below 2^kMtBlkPolys
  // sections; otherwise through the ladder).  kMtUnits: counted in units of
  // 624 2^kMtBlkUnit outputs from the end of the state's block, which is taken
  // as used up (by the digits; fewer than 16^kMtBlkDigits units)
  int mt_blocks = 0;
};

// how the many-stream MRG32K3A/LFSR113 kernels cut and store (regstream.h)
struct RegPlan {
  int nsec_log2 = 0;                  // sections per stream
  uint64_t seclen = 0;
  bool lines = false;                 // sections begin on lines of the output
  uint32_t unit = 128;                // bytes that a run's chunks are aligned to (0: the lanes store by themselves)
  const uint32_t* sectab = nullptr;   // the section-start table of seclen (null: jumps by bytes)
};
hipError_t launch_mrg_generate(const DeviceTables& T, MrgState* states, uint32_t count, uint64_t n, const RegPlan& plan,
                               int dtype, void* out, hipStream_t st);
// one stream cut into sections, a lane each: n outputs of *base (a host
// object, passed by value) to out, the state after them to *sout (device-
// accessible memory)
hipError_t launch_mrg_single(const DeviceTables& T, const MrgState* base, MrgState* sout, uint64_t n, int dtype,
                             void* out, hipStream_t st);
hipError_t launch_lfsr_single(const DeviceTables& T, const LfsrState* base, LfsrState* sout, uint64_t n, int dtype,
                              void* out, hipStream_t st);
// likewise GM/GQ, a wavefront's share each: base and sout device-accessible
// and distinct; wavefronts() of them read the base
hipError_t launch_gm_single(const DeviceTables& T, int gen, const GmState* base, GmState* sout, uint64_t n, int dtype,
                            void* out, hipStream_t st);
uint64_t gm_single_wavefronts(int gen, uint64_t n);
hipError_t launch_mrg_jump(const DeviceTables& T, MrgState* states, uint32_t count, const JumpSpec& js,
                           const MrgState* base, hipStream_t st);

hipError_t launch_lfsr_generate(const DeviceTables& T, LfsrState* states, uint32_t count, uint64_t n,
                                const RegPlan& plan, int dtype, void* out, hipStream_t st);
hipError_t launch_lfsr_jump(const DeviceTables& T, LfsrState* states, uint32_t count, const JumpSpec& js,
                            const LfsrState* base, hipStream_t st);

// n outputs of one stream by `count` sections: the first from *base, `first`
// outputs; the others from states[0 .. count - 2], seclen each, the last one the
// rest; the advanced state to *last
hipError_t launch_mt_sections(const MtState* base, const MtState* states, MtState* last, uint32_t count, uint64_t first,
                              uint64_t seclen, uint64_t n, int dtype, void* out, hipStream_t st);
hipError_t launch_mt_generate(MtState* states, uint32_t count, uint64_t n, int dtype, void* out,
                              hipStream_t st);
hipError_t launch_mt_jump(const DeviceTables& T, MtState* states, uint32_t count, const JumpSpec& js,
                          const MtState* base, hipStream_t st);

hipError_t launch_gm_generate(const DeviceTables& T, int gen, GmState* states, uint32_t count, uint64_t n, int dtype,
                              void* out, hipStream_t st);
hipError_t launch_gm_jump(const DeviceTables& T, int gen, GmState* states, uint32_t count, const JumpSpec& js,
                          const GmState* base, hipStream_t st);

hipError_t launch_seed(int gen, const uint64_t* seeds, uint32_t count, void* states, hipStream_t st);
// the same seeding on the host (no GPU): one state blob of `gen`
void seed_host(int gen, uint64_t seed, void* h_state);

// ---- host-side table construction (context set-up) ----
struct HostTables {
  uint32_t mrg[64 * 256 * 18];
  uint32_t lfsr[kJumpRows * 4 * 32];
  uint64_t gm[8 * kJumpRows * 4];
  uint64_t gmbyte[8 * 8 * 256 * 4];
  uint64_t gmneg[8 * 4];
  GmxTable gmx[8];
  uint32_t lfsrbyte[8 * 256 * 128];
};
void build_mrg_bytes(uint32_t* out);
void build_lfsr_jumps(uint32_t* out);
// Section-start tables of the many-stream MRG32K3A/LFSR113 kernels: for a
// section length L, row j - 1 (j = 1 .. kSectionTableRows) holds the jump by
// j L (MRG32K3A: A^(jL) mod m1 then B^(jL) mod m2, 18 words; LFSR113: the
// columns of T_c^(jL) for c = 0..3, 128 words), so section j of a stream
// starts from one matrix application instead of one per set bit of j L.
constexpr int kSectionTableRows = 63;
constexpr int kMrgSectionWords = 18;
constexpr int kLfsrSectionWords = 128;
void build_mrg_section_table(uint64_t seclen, uint32_t* out);
void build_lfsr_section_table(uint64_t seclen, uint32_t* out);
void build_gm_jumps(uint64_t* out);
void build_gm_byte_tables(uint64_t* out, uint64_t* neg);
void build_gmx_tables(GmxTable* out);
void build_lfsr_byte_table(uint32_t* out);

// the calling thread's current device is set to `dev` for the guard's life
struct DeviceGuard {
  int prev = -1;
  hipError_t err = hipSuccess;
  explicit DeviceGuard(int dev) {
    if (hipGetDevice(&prev) != hipSuccess) prev = -1;
    if (prev != dev) err = hipSetDevice(dev);
  }
  ~DeviceGuard() {
    int cur = -1;
    if (prev >= 0 && hipGetDevice(&cur) == hipSuccess && cur != prev) (void)hipSetDevice(prev);
  }
};

}  // namespace prand

namespace prand {
constexpr size_t kPinBytes = 8192, kPinOut = 4096;
constexpr int kPinSlots = 2;
constexpr size_t kArrayDevBytes = 64u << 20, kArrayPinBytes = 2u << 20;
constexpr int kArrayPins = 3, kArrayKept = 2;

// what one prand_generate_array call works with: a device buffer of up to
// kArrayDevBytes, pinned copy buffers and the events of their copies
struct ArrayBuffers {
  void* dev = nullptr;
  size_t dev_bytes = 0;
  char* pin = nullptr;
  hipEvent_t ev[kArrayPins] = {};
};
static_assert(sizeof(MtState) <= kPinOut, "a state fits half a slot");
}  // namespace prand

// the opaque context of the public ABI
struct prand_ctx {
  int device = 0;
  int num_cus = 256;
  char arch[64] = {0};
  prand::DeviceTables T;
  bool mt_ready = false;
  std::mutex mu;          // guards mt_ready, the host-call scratch and the section buffer
  void* scratch = nullptr;
  // prand_generate's section states and distances, kept between calls and
  // grown when a call needs more (freed with the context)
  void* sec_buf = nullptr;
  size_t sec_buf_bytes = 0;
  int last_hip = 0;
  // pinned host memory: kPinSlots slots of kPinBytes for the states that host
  // calls pass in (at 0) and get back (at kPinOut): slot 0 under mu, slot 1
  // under the allocation-free entry point's lock of the device
  char* pin = nullptr;
  // prand_generate_array: buffers that no call is using, kept between calls (up
  // to kArrayKept sets; a call takes one, or makes its own); arr_mu guards the
  // list alone, calls of several threads run side by side
  std::mutex arr_mu;
  prand::ArrayBuffers* arr_free[prand::kArrayKept] = {};
  // section-start tables by section length, [0] MRG32K3A, [1] LFSR113
  // (built on first use, immutable afterwards, freed with the context)
  std::mutex sec_mu;
  std::vector<std::pair<uint64_t, uint32_t*>> sec_tabs[2];
};

namespace prand {
// build and upload the MT19937 jump polynomials once per context
int ensure_mt_tables(prand_ctx* c);
// whether the MT19937 jump polynomials are built (never builds them)
bool mt_tables_ready(prand_ctx* c);
// the sectioned fill of one host state (prand_generate); with `scratch` set
// it keeps its section states there and allocates nothing
int generate_host_state(prand_ctx* c, int gen, void* h_state, int dtype, void* d_out, uint64_t n,
                        hipStream_t st, void* scratch, size_t scratch_bytes);
// once per device, with that device current: look up the device address of
// the allocation-free entry point's static array
hipError_t noalloc_setup(int device);

inline int hipfail(prand_ctx* c, hipError_t e) {
  if (c) c->last_hip = (int)e;
  return PRAND_EHIP;
}
}  // namespace prand
