// The C ABI declared in include/prand.h: argument checks, context set-up and
// the choice of launch shapes.  Every generated number and every jump is
// computed by the HIP kernels; host code here only validates, plans and
// copies states for the entry points that take host states.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <vector>

#include "mt_poly.h"
#include "prand_impl.h"

using namespace prand;

namespace {

constexpr size_t kScratch = 64 * 1024;

bool valid_gen(int g) { return g >= 0 && g < PRAND_NUM_GENERATORS; }
bool valid_dtype(int d) { return d >= PRAND_U32 && d <= PRAND_F64; }

size_t state_bytes(int g) {
  switch (g) {
    case PRAND_MT19937: return sizeof(MtState);
    case PRAND_MRG32K3A: return sizeof(MrgState);
    case PRAND_LFSR113: return sizeof(LfsrState);
    default: return valid_gen(g) ? sizeof(GmState) : 0;
  }
}
size_t elem_bytes(int dtype) { return dtype == PRAND_F64 ? 8 : 4; }

// Block-splitting block lengths, log2 of ensemble steps, per initialising
// function of the paper's Table 4: the smallest power of two no shorter than
// the table's maximal sequence length.  -1: function not provided.
constexpr int kBlockLog2[PRAND_NUM_GENERATORS][4] = {
    /*            SEQ SHORT MEDIUM LONG */
    /* MT19937  */ {432, -1, -1, -1},
    /* MRG32K3A */ {127, -1, -1, -1},
    /* LFSR113  */ {34, -1, -1, 80},
    /* GM19     */ {23, -1, -1, -1},
    /* GM29     */ {-1, 27, 33, 40},
    /* GM31     */ {-1, 27, 33, 40},
    /* GM55     */ {-1, 34, -1, 67},
    /* GM61     */ {34, -1, -1, 85},
    /* GQ58.1   */ {-1, 27, 33, 40},
    /* GQ58.3   */ {-1, 27, 33, 40},
    /* GQ58.4   */ {-1, 27, 33, 40},
};
// Table 4: (number of sequences, maximal length) per initialising function
constexpr double kLimits[PRAND_NUM_GENERATORS][4][2] = {
    /* MT19937  */ {{1e19, 1e130}, {0, 0}, {0, 0}, {0, 0}},
    /* MRG32K3A */ {{1e19, 1e38}, {0, 0}, {0, 0}, {0, 0}},
    /* LFSR113  */ {{3.8e18, 1e10}, {0, 0}, {0, 0}, {4e9, 1e24}},
    /* GM19     */ {{1e3, 6e6}, {0, 0}, {0, 0}, {0, 0}},
    /* GM29     */ {{0, 0}, {1e8, 8e7}, {1e6, 8e9}, {1e4, 8e11}},
    /* GM31     */ {{0, 0}, {1e9, 8e7}, {1e7, 8e9}, {1e5, 8e11}},
    /* GM55     */ {{0, 0}, {1e18, 1e10}, {0, 0}, {4e9, 1e20}},
    /* GM61     */ {{1.8e19, 1e10}, {0, 0}, {0, 0}, {4e9, 3e25}},
    /* GQ58.1   */ {{0, 0}, {1e8, 8e7}, {1e6, 8e9}, {1e4, 8e11}},
    /* GQ58.3   */ {{0, 0}, {2e8, 8e7}, {2e6, 8e9}, {2e4, 8e11}},
    /* GQ58.4   */ {{0, 0}, {3e8, 8e7}, {3e6, 8e9}, {3e4, 8e11}},
};

// the byte tables are built for each generator's default block exponent
constexpr int default_block_log2(int gen) { return kBlockLog2[gen][0] >= 0 ? kBlockLog2[gen][0] : kBlockLog2[gen][1]; }
constexpr bool byte_tables_match() {
  for (int g = 0; g < 8; g++)
    if (kGmByteE[g] != default_block_log2(PRAND_GM19 + g)) return false;
  return kLfsrByteE == default_block_log2(PRAND_LFSR113);
}
static_assert(byte_tables_match(), "byte tables built for another block exponent");

// the documented default seed of each generator: MT19937 5489, MRG32K3A and
// LFSR113 12345, GM/GQ 0
uint64_t default_seed(int gen) { return gen == PRAND_MT19937 ? 5489 : (gen <= PRAND_LFSR113 ? 12345 : 0); }

int block_log2(int gen, int variant) {
  if (!valid_gen(gen) || variant < PRAND_SEQ_DEFAULT || variant > PRAND_SEQ_LONG) return PRAND_EINVAL;
  if (variant == PRAND_SEQ_DEFAULT) {
    const int e = kBlockLog2[gen][0];
    return e >= 0 ? e : kBlockLog2[gen][1];
  }
  const int e = kBlockLog2[gen][variant - 1];
  return e >= 0 ? e : PRAND_EUNSUPPORTED;
}

int resolve_variant(int gen, int variant) {
  if (variant != PRAND_SEQ_DEFAULT) return variant;
  return kBlockLog2[gen][0] >= 0 ? PRAND_SEQ : PRAND_SEQ_SHORT;
}

template <class T>
hipError_t upload(T** dst, const T* src, size_t n) {
  hipError_t e = hipMalloc((void**)dst, n * sizeof(T));
  if (e != hipSuccess) return e;
  return hipMemcpy(*dst, src, n * sizeof(T), hipMemcpyHostToDevice);
}

// The MT19937 tables (656 MB, read-only once built) are shared by the
// contexts of one device: the first context that needs them builds them, the
// others take references, the last one to go frees them.
struct MtTables {
  uint32_t *mt = nullptr, *mtblk = nullptr, *mtinv = nullptr, *mtdiglo = nullptr, *mtdig8hi = nullptr;
  void* mttop = nullptr;
  int refs = 0;
};
std::mutex g_mt_mu;
std::map<int, MtTables> g_mt_tables;   // by device

void take_mt_tables(prand_ctx* c, const MtTables& t) {
  c->T.mt = t.mt;
  c->T.mtblk = t.mtblk;
  c->T.mtinv = t.mtinv;
  c->T.mtdiglo = t.mtdiglo;
  c->T.mtdig8hi = t.mtdig8hi;
  c->T.mttop = t.mttop;
  c->mt_ready = true;
}

void free_mt_fields(prand_ctx* c) {
  (void)hipFree(c->T.mt);
  (void)hipFree(c->T.mtdiglo);
  (void)hipFree(c->T.mtdig8hi);
  (void)hipFree(c->T.mttop);
  (void)hipFree(c->T.mtblk);
  (void)hipFree(c->T.mtinv);
}

// a context's share of the tables goes (at destruction; its device current)
void release_mt_tables(prand_ctx* c) {
  if (!c->mt_ready) {
    free_mt_fields(c);   // what a failed build left, if anything
    return;
  }
  std::lock_guard<std::mutex> lk(g_mt_mu);
  auto it = g_mt_tables.find(c->device);
  if (it != g_mt_tables.end() && --it->second.refs == 0) {
    free_mt_fields(c);
    g_mt_tables.erase(it);
  }
}

hipError_t ensure_mt(prand_ctx* c) {
  // caller holds c->mu
  if (c->mt_ready) return hipSuccess;
  std::lock_guard<std::mutex> glk(g_mt_mu);
  {
    auto it = g_mt_tables.find(c->device);
    if (it != g_mt_tables.end()) {
      it->second.refs++;
      take_mt_tables(c, it->second);
      return hipSuccess;
    }
  }
  std::vector<uint32_t> mt((size_t)kLadder * 624), dlo((size_t)kMtLoDigits * kMtLoSize * 624),
      d8((size_t)2 * 256 * 624);
  constexpr int kBits = 4 * kMtBlkDigits;
  std::vector<uint32_t> bits((size_t)kBits * 624), blk((size_t)kMtBlkDigits * 16 * 624), inv(624);
  if (!mt_build_polys(mt.data(), kLadder, dlo.data(), d8.data(), kMtDigitE)) return hipErrorUnknown;
  if (!mt_build_block_polys(kMtBlkUnit + kBits + 9, kMtBlkUnit, kBits, bits.data(), inv.data(), blk.data()))
    return hipErrorUnknown;
  hipError_t e = upload(&c->T.mt, mt.data(), mt.size());
  if (e == hipSuccess) e = upload(&c->T.mtblk, blk.data(), blk.size());
  if (e == hipSuccess) e = upload(&c->T.mtinv, inv.data(), inv.size());
  if (e == hipSuccess) e = upload(&c->T.mtdiglo, dlo.data(), dlo.size());
  if (e == hipSuccess) e = upload(&c->T.mtdig8hi, d8.data(), d8.size());
  // the default state jumped t * 2^(432 + 48) for every top-16-bit value t
  // of an id, by the jump kernel's general digit path
  uint64_t* d_ids = nullptr;
  if (e == hipSuccess) e = hipMalloc(&c->T.mttop, (size_t)65536 * sizeof(MtState));
  if (e == hipSuccess) e = hipMalloc((void**)&d_ids, 65536 * sizeof(uint64_t));
  if (e == hipSuccess) {
    std::vector<uint64_t> ids(65536);
    for (uint64_t t = 0; t < 65536; t++) ids[t] = t << 48;
    e = hipMemcpy(d_ids, ids.data(), ids.size() * sizeof(uint64_t), hipMemcpyHostToDevice);
  }
  if (e == hipSuccess) {
    JumpSpec js;
    js.ids = d_ids;
    js.block_e = kMtDigitE;
    e = launch_mt_jump(c->T, (MtState*)c->T.mttop, 65536, js,
                       (const MtState*)((const char*)c->T.defaults + kDefaultStride * PRAND_MT19937), nullptr);
  }
  if (e == hipSuccess) e = hipDeviceSynchronize();
  (void)hipFree(d_ids);
  if (e == hipSuccess) {
    MtTables t;
    t.mt = c->T.mt;
    t.mtblk = c->T.mtblk;
    t.mtinv = c->T.mtinv;
    t.mtdiglo = c->T.mtdiglo;
    t.mtdig8hi = c->T.mtdig8hi;
    t.mttop = c->T.mttop;
    t.refs = 1;
    g_mt_tables[c->device] = t;
    c->mt_ready = true;
  }
  return e;
}

int ensure_mt_locked(prand_ctx* c, int gen) {
  if (gen != PRAND_MT19937) return PRAND_OK;
  std::lock_guard<std::mutex> lk(c->mu);
  hipError_t e = ensure_mt(c);
  return e == hipSuccess ? PRAND_OK : hipfail(c, e);
}

hipError_t launch_jump(prand_ctx* c, int gen, void* states, uint32_t count, const JumpSpec& js, const void* base,
                       hipStream_t st) {
  switch (gen) {
    case PRAND_MT19937: return launch_mt_jump(c->T, (MtState*)states, count, js, (const MtState*)base, st);
    case PRAND_MRG32K3A: return launch_mrg_jump(c->T, (MrgState*)states, count, js, (const MrgState*)base, st);
    case PRAND_LFSR113: return launch_lfsr_jump(c->T, (LfsrState*)states, count, js, (const LfsrState*)base, st);
    default: return launch_gm_jump(c->T, gen, (GmState*)states, count, js, (const GmState*)base, st);
  }
}

// The section-start table of MRG32K3A/LFSR113 (k = 0/1) for section length
// seclen: looked up, or built on the host and uploaded (an allocation and a
// blocking copy, once per length; not while the stream is being captured, and
// at most kMaxSectionTables lengths per generator).
// Null when there is none: the kernel then jumps by the byte tables.
constexpr size_t kMaxSectionTables = 64;

const uint32_t* section_table(prand_ctx* c, int k, uint64_t seclen, hipStream_t st) {
  std::lock_guard<std::mutex> lk(c->sec_mu);
  for (const auto& t : c->sec_tabs[k])
    if (t.first == seclen) return t.second;
  if (c->sec_tabs[k].size() >= kMaxSectionTables) return nullptr;
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(st, &cs) != hipSuccess || cs != hipStreamCaptureStatusNone) return nullptr;
  const size_t words = (size_t)kSectionTableRows * (k == 0 ? kMrgSectionWords : kLfsrSectionWords);
  std::vector<uint32_t> h(words);
  if (k == 0) build_mrg_section_table(seclen, h.data());
  else build_lfsr_section_table(seclen, h.data());
  uint32_t* d = nullptr;
  if (hipMalloc((void**)&d, words * 4) != hipSuccess) {
    (void)hipGetLastError();
    return nullptr;
  }
  if (hipMemcpy(d, h.data(), words * 4, hipMemcpyHostToDevice) != hipSuccess) {
    (void)hipGetLastError();
    (void)hipFree(d);
    return nullptr;
  }
  c->sec_tabs[k].push_back({seclen, d});
  return d;
}

// How a many-stream MRG32K3A/LFSR113 call is cut and stored (regstream.h).
//
// Lanes store by themselves (unit 0) runs of up to 32 bytes, and rows off the
// output's lines that are not much longer while there are few: a frame of chunks
// costs 2 us of set-up and partial rounds (LFSR113, 5574 streams of 9 u32 3.4 us
// so and 6.9 in a frame, of 33 u32 7.0 and 7.6; but 300000 of 9 u32 12.0 and
// 11.6, 33000 of 16 u32 5.9 and 5.4).
//
// few_plan: in a call of up to 10 * 2^20 outputs (f64 or rows on lines: 12) the
// time is the chain of one lane, and the caches join partial lines, so a stream
// is cut into short sections whose starts jump by the byte tables (one matrix per
// nonzero byte of the distance), on 16 bytes and in chunks on 16 bytes; where
// every row is on lines, sections are whole chunks.  Up to 2^16 lanes (while
// they leave SIMDs idle) of 12 outputs or more, on lines 24 (MRG32K3A) and 16,
// where a row is longer than a section's start: from 64 outputs, MRG32K3A from 32
// (LFSR113's matrix, of 128 bits, costs more than 100 outputs, MRG32K3A's 25);
// MRG32K3A also up to 2^19 lanes of 512 bytes (on lines 384).  us, with sections that begin on
// lines wherever the row begins, and so: MRG32K3A 20000 streams of 100 u32 13.7
// and 8.9, 10007 of 1000 26 and 22, of 300 f64 17 and 14; LFSR113 20000 of 100 u32
// 13.9 and 9.6, 10007 of 1000 37 and 27; and with one section per stream, or two
// by the table: MRG32K3A 20000 of 100 u32 10.9, 10007 of 1000 39.
//
// short_plan, of more outputs: short sections that begin on lines, up to 2^16 lanes
// of 16 outputs or more, MRG32K3A up to 2^18 of 128 (20000 streams of 1000 u32
// 35 us, 39 by the table; 10007 of 2500 36 and 44).
// long_plan, where those sections would be longer than 256: starts by a section-start
// table (one matrix), sections of at least 1 KB, as many as fit
// in 2^22 lanes (more, shorter sections measured faster: the 64 runs of a
// wavefront then lie close together in the output; 10007 streams of 4999 f64
// in sections of 2 KB 112 us, of 1 KB 101-109, of u32 in sections of 512 bytes
// 72-74, 75 in those of 1 KB).  LFSR113's start costs as much as a hundred
// outputs: f64 sections have 240 or more where a stream's output is 8 KB at
// most, so that its runs lie together in any case (65536 streams of 600 f64 in
// sections of 150 79 us, of 300 72; but of 5001 545 us in sections of 157, 555
// of 313, and 10007 of 4999 102 and 107).  f64 sections begin on lines, by
// dropping up to 15 outputs (65536 streams of 16383 2.38 ms with partial chunks
// at every section's ends, 1.65 so); u32 and f32 ones do not, as dropping up to
// 31 of 256 costs what it saves (10007 LFSR113 streams of 4999 f32 70 us
// without, 71.5 so).
//
// One section: chunks on 16 bytes for runs of up to a line, and of up to eight
// where the outputs are few (65536 streams of 100 f32 22 us in chunks on 16
// bytes, 24 on lines, of 100 f64 17.3 and 19.9; but 40000 of 250 u32 31.3 and
// 28.8, 300000 of 100 f32 101 and 60).
bool lane_stores(uint32_t count, uint64_t n, uint64_t bytes, bool lines) {
  if (lines || bytes > 272) return false;
  const uint64_t all = count * bytes;
  return bytes < 32 || count <= 128 || (bytes == 32 && all <= (16u << 20)) || (bytes <= 136 && all <= (3u << 19)) ||
         (bytes <= 100 && all <= (bytes % 16 || n <= 8 ? 4u << 20 : 2u << 20));
}
bool few_plan(int gen, uint32_t count, uint64_t n, size_t es, bool lines, RegPlan& p) {
  if (n > (16u << 20) || count * n > (lines || es == 8 ? 12u << 20 : 10u << 20)) return false;
  const bool mrg = gen == PRAND_MRG32K3A;
  const uint64_t least = !lines ? 12 : mrg ? 24 : n <= 64 ? 32 : 16;
  while (p.nsec_log2 < 6 && (lines || n >= (mrg ? 32 : 64))) {
    const uint64_t lanes = (uint64_t)count << (p.nsec_log2 + 1), more = 1ull << (p.nsec_log2 + 1);
    if (!(lanes <= (1u << 16) && n >= least * more) &&
        !(mrg && lanes <= (1u << 19) && n * es >= (lines ? 384 : 512) * more))
      break;
    p.nsec_log2++;
  }
  const uint64_t whole = lines ? 31 : 3;   // sections of whole chunks, or 16-byte pieces
  p.seclen = (((n + (1ull << p.nsec_log2) - 1) >> p.nsec_log2) + whole) & ~whole;
  if (p.nsec_log2 && !lines) {
    p.unit = 16;
    return true;
  }
  return p.seclen <= 256;
}
bool short_plan(int gen, uint32_t count, uint64_t n, bool lines, RegPlan& p) {
  const uint64_t max_lanes = gen == PRAND_MRG32K3A ? 1ull << 18 : 1ull << 16;
  const uint64_t reach = lines ? n : n + 31;   // room to begin the sections on lines
  p.nsec_log2 = 0;
  while (p.nsec_log2 < 6) {
    const uint64_t lanes = (uint64_t)count << (p.nsec_log2 + 1);
    if (lanes > max_lanes || reach >> (p.nsec_log2 + 1) < (lanes <= (1u << 16) ? 16 : 128)) break;
    p.nsec_log2++;
  }
  p.seclen = ((((p.nsec_log2 ? reach : n) + (1ull << p.nsec_log2) - 1) >> p.nsec_log2) + 31) & ~31ull;
  return p.seclen <= 256;
}
void long_plan(int gen, uint32_t count, uint64_t n, int dtype, RegPlan& p) {
  const uint64_t least = gen == PRAND_LFSR113 && dtype == PRAND_F64 && n <= 1024 ? 1920 : 1024;
  p.nsec_log2 = 0;
  while (p.nsec_log2 < 6 && ((uint64_t)count << (p.nsec_log2 + 1)) <= (1ull << 22) &&
         (n >> (p.nsec_log2 + 1)) * elem_bytes(dtype) >= least)
    p.nsec_log2++;
  const uint64_t whole = dtype == PRAND_F64 ? 15 : 31;
  p.seclen = (((n + (1ull << p.nsec_log2) - 1) >> p.nsec_log2) + whole) & ~whole;
}

// many-stream generation, the states moved on in place
hipError_t launch_streams(prand_ctx* c, int gen, void* states, uint32_t count, uint64_t n, int dtype, void* out,
                          hipStream_t st) {
  if (gen == PRAND_MRG32K3A || gen == PRAND_LFSR113) {
    const size_t es = elem_bytes(dtype);
    const bool lines = ((uintptr_t)out | n * es) % 128 == 0;
    RegPlan p;
    p.seclen = n;
    if (lane_stores(count, n, n * es, lines)) {
      p.unit = 0;
    } else if (few_plan(gen, count, n, es, lines, p)) {
      p.lines = lines;
    } else if (short_plan(gen, count, n, lines, p)) {
      p.lines = true;
    } else {
      long_plan(gen, count, n, dtype, p);
      if (p.nsec_log2) p.sectab = section_table(c, gen == PRAND_MRG32K3A ? 0 : 1, p.seclen, st);
      p.lines = dtype == PRAND_F64 || !p.sectab;
    }
    if (p.unit && !p.nsec_log2 && (n * es <= 128 || (n * es <= 1024 && count * n <= (1u << 23)))) p.unit = 16;
    if (gen == PRAND_MRG32K3A) return launch_mrg_generate(c->T, (MrgState*)states, count, n, p, dtype, out, st);
    return launch_lfsr_generate(c->T, (LfsrState*)states, count, n, p, dtype, out, st);
  }
  if (gen == PRAND_MT19937) return launch_mt_generate((MtState*)states, count, n, dtype, out, st);
  return launch_gm_generate(c->T, gen, (GmState*)states, count, n, dtype, out, st);
}

// distances of the section starts: (i + 1) units
__global__ void section_dist_kernel(uint64_t* d, uint32_t count, uint64_t unit) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) d[i] = (i + 1) * unit;
}

// MT19937 outputs that one section makes in no more time than sections with
// their jumps: 200000 u32 80 us, 300000 111; 310000 to 10^6 in sections 103-110
constexpr uint64_t kMtSingle = 1u << 18;

// a state blob between pinned host memory and the device
__global__ void copy_state_kernel(uint32_t* dst, const uint32_t* src, uint32_t words) {
  for (uint32_t i = threadIdx.x; i < words; i += blockDim.x) dst[i] = src[i];
}

void free_array_buffers(ArrayBuffers* b) {
  if (!b) return;
  (void)hipFree(b->dev);
  (void)hipHostFree(b->pin);
  for (hipEvent_t ev : b->ev)
    if (ev) (void)hipEventDestroy(ev);
  delete b;
}

// a set of the context's free ones, or a new one (null: out of memory); given
// back at the end of its scope
struct TakenBuffers {
  prand_ctx* c;
  ArrayBuffers* b = nullptr;
  explicit TakenBuffers(prand_ctx* ctx) : c(ctx) {
    std::lock_guard<std::mutex> lk(c->arr_mu);
    for (ArrayBuffers*& f : c->arr_free)
      if (!b && f) std::swap(b, f);
    if (!b) b = new (std::nothrow) ArrayBuffers;
  }
  ~TakenBuffers() {
    {
      std::lock_guard<std::mutex> lk(c->arr_mu);
      for (ArrayBuffers*& f : c->arr_free)
        if (b && !f) std::swap(b, f);
    }
    free_array_buffers(b);   // more calls at once than sets are kept
  }
};

// the host state in pinned slot 0 after `launch` on it, back to h_state (the
// default stream; the caller holds mu)
template <class F>
int on_host_state(prand_ctx* c, int gen, void* h_state, F&& launch) {
  char* const state = c->pin + kPinOut;
  std::memcpy(state, h_state, state_bytes(gen));
  hipError_t e = launch((void*)state);
  const hipError_t se = hipStreamSynchronize(nullptr);
  if (e == hipSuccess) e = se;
  if (e != hipSuccess) return hipfail(c, e);
  std::memcpy(h_state, state, state_bytes(gen));
  return PRAND_OK;
}

}  // namespace

int prand::ensure_mt_tables(prand_ctx* c) {
  DeviceGuard g(c->device);
  return ensure_mt_locked(c, PRAND_MT19937);
}

// The fill behind prand_generate and prand_generate_noalloc, cut into sections
// that jump to their starts.
//
// MRG32K3A, LFSR113 and GM/GQ: one launch whose lanes or wavefronts jump by
// themselves (a state of 24 or 16 bytes by value, GM/GQ from the pinned slot
// while few wavefronts read it, else from a device copy), the last of which
// leaves the advanced state.
//
// MT19937: one workgroup while one section is enough.  Otherwise sections that
// start on the stream's block boundaries: the first from the state itself, the
// rest of its block and L outputs, section j from the state moved j L outputs
// on from the end of its block (L = 624 * 2^8 * 2^k: a jump per nonzero
// hexadecimal digit of j 2^k), the last one what is left.  A jump yields the
// canonical window, which differs from the array sequential generation holds
// only in bits that the next twist overwrites, and every section begins with a
// twist: the last one's state is exactly the sequential one.  The section
// states, their distances and the copied-in base state live in `scratch` when
// it is given (the plan then uses at most as many sections as fit in
// scratch_bytes; the output does not depend on the plan), else in the
// context's buffers.  (Sections off the boundaries, by the ladder, and one more
// from the last boundary: 10^6 u32 538 us, 110 so; 10^7 650 and 152.)
//
// States come and go through pinned memory that kernels read and write: no
// copy calls.  Arguments are checked by the caller; MT19937 tables must exist.
int prand::generate_host_state(prand_ctx* c, int gen, void* h_state, int dtype, void* d_out, uint64_t n,
                               hipStream_t st, void* scratch, size_t scratch_bytes) {
  const size_t sb = state_bytes(gen);
  const size_t base_bytes = (sb + 255) & ~(size_t)255;
  // base state, then distances, then states, each 256-byte aligned
  if (scratch && scratch_bytes < base_bytes + 2 * 256 + 2 * (sb + 8)) return PRAND_ERANGE;
  std::unique_lock<std::mutex> lk(c->mu, std::defer_lock);
  if (!scratch) lk.lock();
  char* const pin_in = c->pin + (scratch ? kPinBytes : 0);
  char* const pin_out = pin_in + kPinOut;
  std::memcpy(pin_in, h_state, sb);
  std::memcpy(pin_out, h_state, sb);
  hipError_t e = hipSuccess;
  auto finish = [&]() -> int {
    const hipError_t se = hipStreamSynchronize(st);   // also after an error: what was launched uses the slot
    if (e == hipSuccess) e = se;
    if (e != hipSuccess) return hipfail(c, e);
    std::memcpy(h_state, pin_out, sb);
    return PRAND_OK;
  };
  if (gen == PRAND_MRG32K3A) {
    e = launch_mrg_single(c->T, (const MrgState*)h_state, (MrgState*)pin_out, n, dtype, d_out, st);
    return finish();
  }
  if (gen == PRAND_LFSR113) {
    e = launch_lfsr_single(c->T, (const LfsrState*)h_state, (LfsrState*)pin_out, n, dtype, d_out, st);
    return finish();
  }
  // the base state's device copy (without `scratch`: the host calls' scratch)
  void* const d_base = scratch ? scratch : c->scratch;
  const uint32_t words = (uint32_t)(sb / 4);
  if (gen != PRAND_MT19937) {
    const void* base = pin_in;
    if (gm_single_wavefronts(gen, n) > 16) {
      hipLaunchKernelGGL(copy_state_kernel, dim3(1), dim3(256), 0, st, (uint32_t*)d_base, (const uint32_t*)pin_in, words);
      e = hipGetLastError();
      base = d_base;
    }
    if (e == hipSuccess) e = launch_gm_single(c->T, gen, (const GmState*)base, (GmState*)pin_out, n, dtype, d_out, st);
    return finish();
  }
  // up to 512 sections of the shortest length: 80 million outputs
  uint64_t max_secs = 512;
  if (scratch) {
    const uint64_t fit = (scratch_bytes - base_bytes - 2 * 256) / (sb + 8);   // section states that fit
    max_secs = std::min<uint64_t>(max_secs, fit);
  }
  const uint64_t r0 = 624 - std::min<uint32_t>(((const MtState*)h_state)->idx, 624u);
  int k = 0;
  auto seclen = [&]() { return 624ull << (kMtBlkUnit + k); };
  auto sections = [&]() { return n > r0 ? (n - r0 + seclen() - 1) / seclen() : 1; };
  while (sections() > max_secs) k++;
  if (n <= kMtSingle || sections() == 1) {
    // in place in the pinned slot
    e = launch_mt_generate((MtState*)pin_out, 1, n, dtype, d_out, st);
    return finish();
  }
  const uint64_t nst = sections() - 1;   // states: of every section but the first
  void* d_states = nullptr;
  uint64_t* d_dist = nullptr;
  const size_t st_off = (nst * 8 + 255) & ~(size_t)255;
  if (scratch) {
    if (base_bytes + st_off + nst * sb > scratch_bytes) return PRAND_ERANGE;
    d_dist = (uint64_t*)((char*)scratch + base_bytes);
    d_states = (char*)scratch + base_bytes + st_off;
  } else {
    // the context's section buffer (grown when too small, otherwise reused:
    // no allocation and no implicit device synchronisation per call) holds
    // the distances and states
    const size_t need = st_off + nst * sb;
    if (need > c->sec_buf_bytes) {
      (void)hipFree(c->sec_buf);
      c->sec_buf = nullptr;
      c->sec_buf_bytes = 0;
      e = hipMalloc(&c->sec_buf, need);
      if (e == hipSuccess) c->sec_buf_bytes = need;
    }
    if (e == hipSuccess) {
      d_dist = (uint64_t*)c->sec_buf;
      d_states = (char*)c->sec_buf + st_off;
    }
  }
  if (e == hipSuccess) {
    hipLaunchKernelGGL(copy_state_kernel, dim3(1), dim3(256), 0, st, (uint32_t*)d_base, (const uint32_t*)pin_in, words);
    hipLaunchKernelGGL(section_dist_kernel, dim3((uint32_t)((nst + 255) / 256)), dim3(256), 0, st, d_dist,
                       (uint32_t)nst, 1ull << k);
    e = hipGetLastError();
  }
  JumpSpec js;
  js.dist = d_dist;
  js.nlimbs = 1;
  js.per_stream = 1;
  js.mt_blocks = kMtUnits;
  if (e == hipSuccess) e = launch_mt_jump(c->T, (MtState*)d_states, (uint32_t)nst, js, (const MtState*)d_base, st);
  if (e == hipSuccess)
    e = launch_mt_sections((const MtState*)d_base, (const MtState*)d_states, (MtState*)pin_out, (uint32_t)nst + 1,
                           r0 + seclen(), seclen(), n, dtype, d_out, st);
  return finish();
}

bool prand::mt_tables_ready(prand_ctx* c) {
  std::lock_guard<std::mutex> lk(c->mu);
  return c->mt_ready;
}

extern "C" {

const char* prand_strerror(int code) {
  switch (code) {
    case PRAND_OK: return "success";
    case PRAND_EINVAL: return "invalid argument";
    case PRAND_EUNSUPPORTED: return "variant not provided for this generator";
    case PRAND_ERANGE: return "size out of range";
    case PRAND_EHIP: return "HIP runtime error";
    case PRAND_ENOMEM: return "out of memory";
    case PRAND_ENODEV: return "no usable gfx950 device";
    case PRAND_EBUSY: return "request queue full";
    case PRAND_ENOTREADY: return "context tables this call needs are not built yet";
    default: return "unknown error";
  }
}

int prand_last_hip_error(const prand_ctx* ctx) { return ctx ? ctx->last_hip : 0; }

size_t prand_state_bytes(int gen) { return state_bytes(gen); }

int prand_block_log2(int gen, int variant) { return block_log2(gen, variant); }

int prand_independence_limit(int gen, int variant, double* max_streams, double* max_length) {
  const int e = block_log2(gen, variant);
  if (e < 0) return e;
  if (!max_streams || !max_length) return PRAND_EINVAL;
  const int v = resolve_variant(gen, variant) - 1;
  *max_streams = kLimits[gen][v][0];
  *max_length = kLimits[gen][v][1];
  return PRAND_OK;
}

int prand_ctx_create(prand_ctx** out, int hip_device) {
  if (!out) return PRAND_EINVAL;
  *out = nullptr;
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess || hip_device < 0 || hip_device >= ndev) return PRAND_ENODEV;
  hipDeviceProp_t prop;
  if (hipGetDeviceProperties(&prop, hip_device) != hipSuccess) return PRAND_ENODEV;
  if (std::strncmp(prop.gcnArchName, "gfx950", 6) != 0) return PRAND_ENODEV;
  DeviceGuard g(hip_device);
  if (g.err != hipSuccess) return PRAND_ENODEV;
  prand_ctx* c = new (std::nothrow) prand_ctx;
  if (!c) return PRAND_ENOMEM;
  c->device = hip_device;
  c->num_cus = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 256;
  std::strncpy(c->arch, prop.gcnArchName, sizeof(c->arch) - 1);
  HostTables* H = new (std::nothrow) HostTables;
  if (!H) { delete c; return PRAND_ENOMEM; }
  build_mrg_bytes(H->mrg);
  build_lfsr_jumps(H->lfsr);
  build_gm_jumps(H->gm);
  build_gm_byte_tables(H->gmbyte, H->gmneg);
  build_lfsr_byte_table(H->lfsrbyte);
  build_gmx_tables(H->gmx);
  hipError_t e = upload(&c->T.mrg, H->mrg, sizeof(H->mrg) / sizeof(H->mrg[0]));
  if (e == hipSuccess) e = upload(&c->T.lfsr, H->lfsr, sizeof(H->lfsr) / sizeof(H->lfsr[0]));
  if (e == hipSuccess) e = upload(&c->T.gm, H->gm, sizeof(H->gm) / sizeof(H->gm[0]));
  if (e == hipSuccess) e = upload(&c->T.gmbyte, H->gmbyte, sizeof(H->gmbyte) / sizeof(H->gmbyte[0]));
  if (e == hipSuccess) e = upload(&c->T.gmneg, H->gmneg, sizeof(H->gmneg) / sizeof(H->gmneg[0]));
  if (e == hipSuccess) e = upload(&c->T.gmx, H->gmx, sizeof(H->gmx) / sizeof(H->gmx[0]));
  if (e == hipSuccess) e = upload(&c->T.lfsrbyte, H->lfsrbyte, sizeof(H->lfsrbyte) / sizeof(H->lfsrbyte[0]));
  delete H;
  if (e == hipSuccess) e = hipMalloc(&c->T.defaults, kDefaultStride * PRAND_NUM_GENERATORS);
  if (e == hipSuccess) e = hipMalloc(&c->scratch, kScratch);
  if (e == hipSuccess) e = hipHostMalloc((void**)&c->pin, kPinSlots * kPinBytes, hipHostMallocMapped);
  if (e == hipSuccess) e = noalloc_setup(hip_device);
  if (e == hipSuccess) {
    // default states: the documented default seed of each generator
    uint64_t seeds[PRAND_NUM_GENERATORS];
    for (int gidx = 0; gidx < PRAND_NUM_GENERATORS; gidx++)
      seeds[gidx] = default_seed(gidx);
    e = hipMemcpy(c->scratch, seeds, sizeof seeds, hipMemcpyHostToDevice);
    for (int gidx = 0; gidx < PRAND_NUM_GENERATORS && e == hipSuccess; gidx++)
      e = launch_seed(gidx, (const uint64_t*)c->scratch + gidx, 1, (char*)c->T.defaults + kDefaultStride * gidx,
                      nullptr);
    if (e == hipSuccess) e = hipDeviceSynchronize();
  }
  if (e != hipSuccess) {
    prand_ctx_destroy(c);
    return PRAND_EHIP;
  }
  *out = c;
  return PRAND_OK;
}

int prand_ctx_destroy(prand_ctx* c) {
  if (!c) return PRAND_OK;
  DeviceGuard g(c->device);
  (void)hipDeviceSynchronize();
  (void)hipFree(c->T.mrg);
  (void)hipFree(c->T.lfsr);
  (void)hipFree(c->T.gm);
  (void)hipFree(c->T.gmbyte);
  (void)hipFree(c->T.gmneg);
  (void)hipFree(c->T.gmx);
  (void)hipFree(c->T.lfsrbyte);
  release_mt_tables(c);
  (void)hipFree(c->T.defaults);
  (void)hipFree(c->scratch);
  (void)hipFree(c->sec_buf);
  (void)hipHostFree(c->pin);
  for (ArrayBuffers* b : c->arr_free) free_array_buffers(b);
  for (auto& v : c->sec_tabs)
    for (auto& t : v) (void)hipFree(t.second);
  delete c;
  return PRAND_OK;
}

int prand_seed_dev(prand_ctx* c, int gen, const uint64_t* d_seeds, uint32_t count, void* d_states, void* stream) {
  if (!c || !valid_gen(gen)) return PRAND_EINVAL;
  if (count == 0) return PRAND_OK;
  if (!d_seeds || !d_states) return PRAND_EINVAL;
  DeviceGuard g(c->device);
  hipError_t e = launch_seed(gen, d_seeds, count, d_states, (hipStream_t)stream);
  return e == hipSuccess ? PRAND_OK : hipfail(c, e);
}

int prand_seed(prand_ctx* c, int gen, uint64_t seed, void* h_state) {
  if (!c || !valid_gen(gen) || !h_state) return PRAND_EINVAL;
  DeviceGuard g(c->device);
  std::lock_guard<std::mutex> lk(c->mu);
  std::memcpy(c->pin, &seed, 8);
  return on_host_state(c, gen, h_state,
                       [&](void* state) { return launch_seed(gen, (const uint64_t*)c->pin, 1, state, nullptr); });
}

int prand_seed_host(int gen, uint64_t seed, void* h_state) {
  if (!valid_gen(gen) || !h_state) return PRAND_EINVAL;
  seed_host(gen, seed, h_state);
  return PRAND_OK;
}

int prand_init_default_host(int gen, void* h_state) {
  if (!valid_gen(gen) || !h_state) return PRAND_EINVAL;
  seed_host(gen, default_seed(gen), h_state);
  return PRAND_OK;
}

int prand_init_default(prand_ctx* c, int gen, void* h_state) {
  if (!c || !valid_gen(gen) || !h_state) return PRAND_EINVAL;
  DeviceGuard g(c->device);
  hipError_t e = hipMemcpy(h_state, (char*)c->T.defaults + kDefaultStride * gen, state_bytes(gen),
                           hipMemcpyDeviceToHost);
  return e == hipSuccess ? PRAND_OK : hipfail(c, e);
}

// Not in the public header (a test hook): jumps `count` MT19937 states by
// d_sections[i] whole sections of 624 * 2^kMtBlkFirst outputs each, the way
// the serving loop starts its sections (the whole-block table from a block
// boundary and below 2^kMtBlkPolys sections, the ladder otherwise).
int prand_internal_mt_jump_sections(prand_ctx* c, void* d_states, uint32_t count, const uint64_t* d_sections,
                                    void* stream) {
  if (!c) return PRAND_EINVAL;
  if (count == 0) return PRAND_OK;
  if (!d_states || !d_sections) return PRAND_EINVAL;
  DeviceGuard g(c->device);
  int rc = ensure_mt_locked(c, PRAND_MT19937);
  if (rc) return rc;
  JumpSpec js;
  js.dist = d_sections;
  js.nlimbs = 1;
  js.per_stream = 1;
  js.mt_blocks = kMtSections;
  hipError_t e = launch_mt_jump(c->T, (MtState*)d_states, count, js, nullptr, (hipStream_t)stream);
  return e == hipSuccess ? PRAND_OK : hipfail(c, e);
}

// Not in the public header (a test hook): the ranges in which a launch over
// `count` streams goes out (launch_ranges); returns their number, the first
// `max` of them in ranges[3 i ..]: first stream, streams, workgroups.
int prand_internal_launch_ranges(uint64_t count, uint32_t block, uint32_t per_block, uint64_t* ranges, int max) {
  int k = 0;
  (void)launch_ranges(count, block, per_block, [&](uint64_t first, uint32_t m, uint32_t blocks) {
    if (k < max) {
      ranges[3 * k] = first;
      ranges[3 * k + 1] = m;
      ranges[3 * k + 2] = blocks;
    }
    k++;
    return hipSuccess;
  });
  return k;
}

int prand_skipahead_dev(prand_ctx* c, int gen, void* d_states, uint32_t count, const uint64_t* d_dist, int nlimbs,
                        int per_stream, void* stream) {
  if (!c || !valid_gen(gen) || nlimbs < 0 || nlimbs > kMaxLimbs) return PRAND_EINVAL;
  if (count == 0 || nlimbs == 0) return PRAND_OK;
  if (!d_states || !d_dist) return PRAND_EINVAL;
  DeviceGuard g(c->device);
  int rc = ensure_mt_locked(c, gen);
  if (rc) return rc;
  JumpSpec js;
  js.dist = d_dist;
  js.nlimbs = nlimbs;
  js.per_stream = per_stream ? 1 : 0;
  hipError_t e = launch_jump(c, gen, d_states, count, js, nullptr, (hipStream_t)stream);
  return e == hipSuccess ? PRAND_OK : hipfail(c, e);
}

int prand_skipahead(prand_ctx* c, int gen, void* h_state, const uint64_t* h_dist, int nlimbs) {
  if (!c || !valid_gen(gen) || !h_state || nlimbs < 0 || nlimbs > kMaxLimbs || (nlimbs > 0 && !h_dist))
    return PRAND_EINVAL;
  if (nlimbs == 0) return PRAND_OK;
  DeviceGuard g(c->device);
  int rc = ensure_mt_locked(c, gen);
  if (rc) return rc;
  std::lock_guard<std::mutex> lk(c->mu);
  std::memcpy(c->pin, h_dist, 8 * (size_t)nlimbs);
  JumpSpec js;
  js.dist = (const uint64_t*)c->pin;
  js.nlimbs = nlimbs;
  return on_host_state(c, gen, h_state,
                       [&](void* state) { return launch_jump(c, gen, state, 1, js, nullptr, nullptr); });
}

int prand_init_streams_dev(prand_ctx* c, int gen, int variant, const void* d_base_state, const uint64_t* d_ids,
                           uint32_t count, void* d_states, void* stream) {
  if (!c || !valid_gen(gen)) return PRAND_EINVAL;
  const int be = block_log2(gen, variant);
  if (be < 0) return be;
  if (count == 0) return PRAND_OK;
  if (!d_ids || !d_states) return PRAND_EINVAL;
  DeviceGuard g(c->device);
  int rc = ensure_mt_locked(c, gen);
  if (rc) return rc;
  JumpSpec js;
  js.ids = d_ids;
  js.block_e = be;
  const void* base = d_base_state ? d_base_state : (const char*)c->T.defaults + kDefaultStride * gen;
  if (!d_base_state && gen == PRAND_MT19937) js.mt_top = c->T.mttop;
  hipError_t e = launch_jump(c, gen, d_states, count, js, base, (hipStream_t)stream);
  return e == hipSuccess ? PRAND_OK : hipfail(c, e);
}

int prand_init_stream(prand_ctx* c, int gen, int variant, uint64_t id, void* h_state) {
  if (!c || !valid_gen(gen) || !h_state) return PRAND_EINVAL;
  const int be = block_log2(gen, variant);
  if (be < 0) return be;
  DeviceGuard g(c->device);
  int rc = ensure_mt_locked(c, gen);
  if (rc) return rc;
  std::lock_guard<std::mutex> lk(c->mu);
  std::memcpy(c->pin, &id, 8);
  JumpSpec js;
  js.ids = (const uint64_t*)c->pin;
  js.block_e = be;
  if (gen == PRAND_MT19937) js.mt_top = c->T.mttop;
  return on_host_state(c, gen, h_state, [&](void* state) {
    return launch_jump(c, gen, state, 1, js, (const char*)c->T.defaults + kDefaultStride * gen, nullptr);
  });
}

int prand_generate_array(prand_ctx* c, int gen, void* h_state, int dtype, void* h_out, uint64_t n) {
  if (!c || !valid_gen(gen) || !valid_dtype(dtype) || !h_state) return PRAND_EINVAL;
  if (n == 0) return PRAND_OK;
  if (!h_out) return PRAND_EINVAL;
  if (n > (1ull << 40)) return PRAND_ERANGE;
  DeviceGuard g(c->device);
  int rc = ensure_mt_locked(c, gen);
  if (rc) return rc;
  // Chunks of up to kArrayDevBytes: each is filled on the device by the
  // sectioned fill (which continues the host state) and goes to the host
  // array by way of pinned buffers, one piece copied from the device while the
  // CPU copies the one before on: 10^7 MRG32K3A f32 took 2.4 ms by one copy
  // into pageable memory, 1.5 so (the copying CPU's rate, 27 GB/s).  A call of
  // at most 256 KB is generated straight into a pinned buffer.
  TakenBuffers taken(c);
  ArrayBuffers* const b = taken.b;
  if (!b) return PRAND_ENOMEM;
  const size_t es = elem_bytes(dtype);
  hipError_t e = hipSuccess;
  if (!b->pin) {
    e = hipHostMalloc((void**)&b->pin, kArrayPins * kArrayPinBytes, hipHostMallocMapped);
    if (e != hipSuccess) b->pin = nullptr;
  }
  for (hipEvent_t& ev : b->ev)
    if (e == hipSuccess && !ev) e = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
  const uint64_t chunk = std::min<uint64_t>(n, kArrayDevBytes / es);
  const bool direct = n * es <= (256u << 10);
  if (e == hipSuccess && !direct && b->dev_bytes < chunk * es) {
    (void)hipFree(b->dev);
    b->dev = nullptr;
    b->dev_bytes = 0;
    e = hipMalloc(&b->dev, chunk * es);
    if (e == hipSuccess) b->dev_bytes = chunk * es;
  }
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return e == hipErrorOutOfMemory ? PRAND_ENOMEM : hipfail(c, e);
  }
  if (direct) {
    rc = generate_host_state(c, gen, h_state, dtype, b->pin, n, nullptr, nullptr, 0);
    if (rc == PRAND_OK) std::memcpy(h_out, b->pin, n * es);
    return rc;
  }
  for (uint64_t done = 0; done < n && rc == PRAND_OK; done += chunk) {
    const uint64_t m = std::min(chunk, n - done);
    rc = generate_host_state(c, gen, h_state, dtype, b->dev, m, nullptr, nullptr, 0);
    if (rc != PRAND_OK) break;
    const size_t bytes = m * es, pieces = (bytes + kArrayPinBytes - 1) / kArrayPinBytes;
    char* const to = (char*)h_out + done * es;
    auto size_of = [&](size_t k) { return std::min(kArrayPinBytes, bytes - k * kArrayPinBytes); };
    auto start = [&](size_t k) {
      if (e == hipSuccess)
        e = hipMemcpyAsync(b->pin + (k % kArrayPins) * kArrayPinBytes, (char*)b->dev + k * kArrayPinBytes,
                           size_of(k), hipMemcpyDeviceToHost, nullptr);
      if (e == hipSuccess) e = hipEventRecord(b->ev[k % kArrayPins], nullptr);
    };
    for (size_t k = 0; k < std::min<size_t>(pieces, kArrayPins); k++) start(k);
    for (size_t k = 0; k < pieces && e == hipSuccess; k++) {
      e = hipEventSynchronize(b->ev[k % kArrayPins]);
      if (e != hipSuccess) break;
      std::memcpy(to + k * kArrayPinBytes, b->pin + (k % kArrayPins) * kArrayPinBytes, size_of(k));
      if (k + kArrayPins < pieces) start(k + kArrayPins);
    }
    if (e != hipSuccess) {
      (void)hipDeviceSynchronize();   // no copy may outlive the call
      rc = hipfail(c, e);
    }
  }
  return rc;
}

int prand_generate_streams(prand_ctx* c, int gen, void* d_states, uint32_t count, uint64_t n, int dtype,
                           void* d_out, void* stream) {
  if (!c || !valid_gen(gen) || !valid_dtype(dtype)) return PRAND_EINVAL;
  if (count == 0 || n == 0) return PRAND_OK;
  if (!d_states || !d_out) return PRAND_EINVAL;
  if (n > (1ull << 40) || (unsigned __int128)count * n * elem_bytes(dtype) > ((unsigned __int128)1 << 50))
    return PRAND_ERANGE;
  DeviceGuard g(c->device);
  hipError_t e = launch_streams(c, gen, d_states, count, n, dtype, d_out, (hipStream_t)stream);
  return e == hipSuccess ? PRAND_OK : hipfail(c, e);
}

int prand_generate(prand_ctx* c, int gen, void* h_state, int dtype, void* d_out, uint64_t n, void* stream) {
  if (!c || !valid_gen(gen) || !valid_dtype(dtype) || !h_state) return PRAND_EINVAL;
  if (n == 0) return PRAND_OK;
  if (!d_out) return PRAND_EINVAL;
  if (n > (1ull << 40)) return PRAND_ERANGE;
  DeviceGuard g(c->device);
  int rc = ensure_mt_locked(c, gen);
  if (rc) return rc;
  return generate_host_state(c, gen, h_state, dtype, d_out, n, (hipStream_t)stream, nullptr, 0);
}

}  // extern "C"
