// gspar: gradient sparsification (Wangni, Wang, Liu, Zhang; arXiv 1710.09854) for MI355X / gfx950.
//
// Pipeline per call (all launches on the caller's stream, no host synchronisation). The streaming
// passes hand over to the next kernel at its boundary, because device-scope fences are expensive on
// a multi-XCD part.
//   k_init     clears the per-call workspace and writes each row's budget B = rho*d (for a
//              segmented call, one row per segment, also the maps that give each workgroup of the
//              later passes its segment, so that only workgroups holding coordinates are launched).
//   k_stats    one streaming pass over g: an LDS histogram over binades of the magnitude bit pattern
//              (count, exact significand sum, max), added into per-row global copies.
//   k_solve    the solver (Proposition 1; Algorithm 2's criterion with a density budget or as
//              printed, or Algorithm 3): a leading workgroup per row sums the copies and decides;
//              where a threshold cuts a binade that holds several keys, the row's workgroups list,
//              bin or count that binade's keys for it, down to single bit patterns, so every
//              threshold the solvers need is resolved exactly.
//   k_sample   one streaming pass: Philox4x32-10 per group of four coordinates, Bernoulli selection,
//              amplification to g_i or sign(g_i)/lambda, order-preserving compaction with a
//              decoupled look-back across tiles.
//   k_probs    (probabilities entry points) writes p_i = min(lambda |g_i|, 1); k_probs_out writes
//              the per-row results.
// Separately, k_aggregate averages M workers' sparse lists into one dense vector (Algorithm 1,
// step 6), summing each coordinate in fp64 in worker order.
//
// Sums of magnitudes are exact: a magnitude's bit pattern (its "key") fixes its binade, bins never
// straddle a binade, so per-bin sums of 24-bit significands are exact integers and are combined
// in a fixed-point sum (unit 2^-149) that is rounded once to double. Hence lambda, the capped set
// and every decision are independent of the launch geometry and of atomic order.
#include <hip/hip_runtime.h>

#include <climits>
#include <algorithm>
#include <mutex>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <type_traits>

#include "gspar.h"
#ifdef GSPAR_INSTRUMENT
#include <hip/hip_ext.h>

#include "gspar_instr.h"
#endif

#define GS_HD __host__ __device__ __forceinline__

namespace gspar {

constexpr uint32_t kKeyInf = 0x7F800000u;   // bit pattern of +inf: keys >= this are non-finite
constexpr int kNT = 512;                    // threads of the histogram / solver workgroups
constexpr int kLaneCopies = 8;              // LDS copies of the statistics histogram (by lane)
constexpr int kC1 = 4;                      // global copies of the level-1 histogram per row
constexpr int kB1 = 256;                    // level 1: one bin per binade (key >> 23)
constexpr int kWB = 512;                    // bins of a refinement window, one per thread
constexpr int kWC = 4;                      // copies of a window, in LDS by lane and in global memory
static_assert(kWB == kNT, "one bin per thread");
constexpr int kTileThreads = 256;
constexpr int kTileGroups = 16;             // float4 groups per thread per tile
constexpr int kTileElems = kTileThreads * kTileGroups * 4;  // 16384 coordinates per tile
// Sample tiles resident at once (256 CUs x 7); larger grids give each workgroup two tiles (a build
// may lower the threshold to exercise that path on small inputs).
#ifndef GSPAR_SAMPLE_RESIDENT
#define GSPAR_SAMPLE_RESIDENT (256 * 7)
#endif
constexpr int64_t kSampleResident = GSPAR_SAMPLE_RESIDENT;
constexpr int kMaxIters = 64;
constexpr int64_t kMaxChunk = (1 << 20) - 4;  // LDS packing holds < 2^20 elements per workgroup
static_assert(INT32_MAX / kMaxChunk + 1 <= 2049, "histogram chunks of the longest row");

enum : uint32_t { kFlagInternal = 16 };

// ------------------------------------------------------------------------------------------
// Exact sums. A value v * 2^s is added into an array of 32-bit digits held in 64-bit words (digit i
// weighs 2^(32 i)); a word takes up to 2^30 additions before it could overflow, so many threads can
// add with plain 64-bit atomics and no carry, and the carries are resolved once, when the sum is
// rounded. Magnitudes are in units of 2^-149 (the smallest subnormal float), their squares in units
// of 2^-298.
// ------------------------------------------------------------------------------------------
constexpr int kDig = 11;    // sums of magnitudes: below 2^31 * 2^24 * 2^254 = 2^309
constexpr int kDigSq = 20;  // sums of squares: below 2^31 * 2^48 * 2^508 = 2^587

// The three digit additions of v * 2^s, s in [0, smax]: x[i] goes to digit at + i. A shift outside
// the range breaks an invariant of the callers (a binade index outside [0, 255]) and is reported:
// kFlagInternal, and nothing to add.
GS_HD uint32_t dig_split(uint64_t v, int s, int smax, int& at, uint64_t x[3]) {
  const bool ok = s >= 0 && s <= smax;
  at = ok ? s >> 5 : 0;
  const int off = s & 31;
  const uint64_t a = (v & 0xFFFFFFFFull) << off, b = (v >> 32) << off;
  x[0] = ok ? a & 0xFFFFFFFFull : 0;
  x[1] = ok ? (a >> 32) + (b & 0xFFFFFFFFull) : 0;
  x[2] = ok ? b >> 32 : 0;
  return ok ? 0u : (uint32_t)kFlagInternal;
}

// Rounds the digit sum times 2^unit to the nearest double, ties to even: the top 64 bits with every
// lower bit folded into the last one, then two exact conversions and one rounded addition.
template <int N, class T>
GS_HD double dig_round(const T* d, int unit) {
  uint64_t carry = 0, next = d[0];
  uint32_t p1 = 0, p2 = 0, low = 0;          // the digits below the current one, and all below those
  uint32_t t0 = 0, t1 = 0, t2 = 0, rest = 0;  // the same at the highest nonzero digit
  int top = 0;
#pragma unroll 1
  for (int i = 0; i < N; ++i) {
    const uint64_t v = next + carry;
    next = d[i + 1 < N ? i + 1 : i];
    const uint32_t x = (uint32_t)v;
    carry = v >> 32;
    if (x) {
      top = i;
      t0 = x;
      t1 = p1;
      t2 = p2;
      rest = low;
    }
    low |= p2;
    p2 = p1;
    p1 = x;
  }
  if (t0 == 0) return 0.0;
  const int lz = __builtin_clz(t0);
  uint64_t m = (((uint64_t)t0 << 32) | t1) << lz;
  m |= lz ? t2 >> (32 - lz) : 0u;
  m |= ((t2 << lz) | rest) != 0 ? 1u : 0u;
  return ldexp((double)(uint32_t)(m >> 32) * 0x1p32 + (double)(uint32_t)m, 32 * (top - 1) - lz + unit);
}

// ------------------------------------------------------------------------------------------
// Magnitude keys.
// ------------------------------------------------------------------------------------------
GS_HD uint32_t key_of(float x) {
  uint32_t u;
  memcpy(&u, &x, 4);
  return u & 0x7FFFFFFFu;
}
GS_HD double key_value(uint32_t k) {
  float f;
  memcpy(&f, &k, 4);
  return (double)f;
}
GS_HD uint64_t key_sig(uint32_t key) {  // integer significand: value = sig * 2^(max(e,1) - 150)
  uint32_t e = key >> 23, m = key & 0x7FFFFFu;
  return e ? (uint64_t)(m | 0x800000u) : (uint64_t)m;
}
GS_HD int binade_shift(int e) { return (e > 0 ? e : 1) - 1; }  // in units of 2^-149

// Smallest key t with fl(lambda * value(t)) >= 1, i.e. capped <=> key >= t for p = min(lambda a, 1).
// kKeyInf when no finite magnitude is capped.
GS_HD uint32_t cap_key(double lam) {
  if (!(lam > 0.0)) return kKeyInf;
  if (lam == INFINITY) return 1;
  double x = 1.0 / lam;
  uint32_t k;
  if (x >= 3.4028234663852886e38) {
    k = kKeyInf;
  } else {
    k = key_of((float)x);
    if (k == 0) k = 1;
  }
#pragma unroll 1
  for (int it = 0; it < 4 && k > 1 && lam * key_value(k - 1) >= 1.0; ++it) --k;
#pragma unroll 1
  for (int it = 0; it < 4 && k < kKeyInf && !(lam * key_value(k) >= 1.0); ++it) ++k;
  return k;
}

// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11): ten rounds of two 32x32->64 products on
// counter words 0 and 2, high halves crossed with words 1, 3 and the round key; the key advances
// by the golden-ratio and sqrt(3)-1 Weyl increments after each round.
// a ^ b ^ c (one three-input bitwise instruction on gfx950)
GS_HD uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
#else
  return a ^ b ^ c;
#endif
}

GS_HD void philox10(uint32_t& c0, uint32_t& c1, uint32_t& c2, uint32_t& c3, uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    uint64_t m0 = (uint64_t)c0 * 0xD2511F53u;
    uint64_t m1 = (uint64_t)c2 * 0xCD9E8D57u;
    uint32_t x0 = xor3((uint32_t)(m1 >> 32), c1, k0);
    uint32_t x2 = xor3((uint32_t)(m0 >> 32), c3, k1);
    c1 = (uint32_t)m1;
    c3 = (uint32_t)m0;
    c0 = x0;
    c2 = x2;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
}

// ------------------------------------------------------------------------------------------
// Workspace.
// ------------------------------------------------------------------------------------------
// A row's control block. The first 128 bytes are the solver's hand-off words, read and written by
// its workgroups at agent scope while the solver kernel runs; the rest is written by one kernel and
// read by later ones.
struct alignas(256) RowCtl {
  uint64_t req;      // the current request (see Pass; 0: none yet)
  uint32_t lcount;   // keys in the list (kReqList)
  uint32_t pad0[29];
  double B;          // rho * d (the variance-budget solver: eps)
  double lam;        // lambda of Proposition 1
  float inv_lam;     // fl32(1/lambda): the amplified value off the capped set
  uint32_t tcap;     // coordinate capped (p = 1) iff key >= tcap
  uint32_t flags;
  uint32_t done;     // 1 once lambda and tcap are final
  int32_t solver;
  int32_t T;
  uint32_t pad1[6];
  uint32_t src;      // 1: the solver's last request read the candidates
  uint32_t pad2[6];
  uint32_t band_lo;  // candidate band [band_lo, band_hi) of keys (whole binades) the statistics pass
  uint32_t band_hi;  // collected, written by its first workgroup (equal bounds: no band)
  uint32_t pad3;
  uint64_t cand_n;   // candidates collected (above the capacity: incomplete, unused)
  uint64_t pad4[2];
};
static_assert(sizeof(RowCtl) == 256, "RowCtl layout");
// offsets read by the tests to see which source a refinement pass used
static_assert(offsetof(RowCtl, B) == 128 && offsetof(RowCtl, src) == 192 && offsetof(RowCtl, band_lo) == 220 &&
                  offsetof(RowCtl, band_hi) == 224 && offsetof(RowCtl, cand_n) == 232,
              "RowCtl offsets known to the tests");

struct Hist1 {
  uint64_t cnt[kB1];
  uint64_t sig[kB1];
  uint32_t mx[kB1];
};
// Variance-budget solver: squared significands m^2 < 2^48 of the level-1 histogram copies, summed as
// their bits 24-47 (qh) and 0-23 (ql).
struct H1Q {
  uint64_t qh[kB1];
  uint64_t ql[kB1];
};
// One copy of a refinement window: per bin the count, the maximum key's offset in the window, and the
// sums of the offsets within the bin and (variance budget) of their squares.
struct WinBins {
  uint32_t cnt[kWB];
  uint32_t mx[kWB];
  uint64_t sr[kWB];
  uint64_t s2[kWB];
};
// The solver's scratch of a row: copies of the refinement window and the list of the keys of a
// range, when it holds few enough.
constexpr size_t kScratchBytes = 345856;
constexpr int kMaxChunks = 2048 + 8;  // histogram chunks of the longest row (2^31 - 1 coordinates)
// A chunk of the row's requests: the last request that was taken and that was finished, and for
// kReqCount its keys >= qkey and their significand sum.
struct ChunkState {
  uint32_t taken;
  uint32_t done;
  uint32_t qcnt;
  uint32_t pad;
  uint64_t qsig;
};
constexpr int kListMax =
    (int)((kScratchBytes - kWC * sizeof(WinBins) - kMaxChunks * sizeof(ChunkState)) / sizeof(uint32_t));
// Keys of a range up to which it is listed instead of binned again (a build may lower it to exercise
// the windows on small inputs).
#ifndef GSPAR_LIST_CAP
#define GSPAR_LIST_CAP kListMax
#endif
constexpr uint32_t kListCap = GSPAR_LIST_CAP;
struct alignas(256) RowScratch {
  WinBins win[kWC];
  ChunkState chunk[kMaxChunks];
  uint32_t list[kListMax];
};
static_assert(sizeof(RowScratch) == kScratchBytes && kListCap <= (uint32_t)kListMax, "solver scratch of a row");

// Per-row partial count of capped coordinates written by the probabilities pass, one per class.
struct alignas(128) CountLine {
  unsigned long long v;
  unsigned long long pad[15];
};

// Per-row histogram over binades of a systematic sample of the row (count and significand sum),
// from which every statistics workgroup predicts the band of keys the solvers will refine.
struct PreHist {
  uint64_t cnt[kB1];
  uint64_t sig[kB1];
};

GS_HD size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

struct Layout {
  size_t ctl, h1, scratch, kc, status, bmap, tmap, h1q, pre, ccnt, cand, total;
  int64_t tiles;     // tiles per row of the sample pass
  int64_t cand_cap;  // candidate keys per row (0: no candidate band)
};

constexpr int64_t kMinChunk = 8192;  // fewest coordinates per histogram workgroup (but the row's)

// Candidate band: rows of at least kCandMinRow coordinates predict, from a sample of the row, the
// binades holding every threshold the solvers will refine, and the statistics pass copies the keys
// inside them to a per-row buffer, so refinement passes read those keys instead of the row. The
// sample costs a launch (about 5 us) and the collection a few per cent of the statistics pass, a
// loss on rows whose passes over the row take about as long or that need no window at all, so
// only rows of 2^25 coordinates and more take the band (a build may lower the threshold to
// exercise the band on small inputs).
#ifndef GSPAR_CAND_MIN_ROW
#define GSPAR_CAND_MIN_ROW (1 << 25)
#endif
constexpr int64_t kCandMinRow = GSPAR_CAND_MIN_ROW;
static_assert(kCandMinRow >= 1024, "a row must hold at least 64 whole lines to be sampled");
constexpr int kPreWG = 64;              // sample workgroups per row
#ifndef GSPAR_PRE_LINES
#define GSPAR_PRE_LINES 256
#endif
constexpr int kPreLines = GSPAR_PRE_LINES;  // 64-byte lines sampled per workgroup (16384 per row)
// Lines of a row of length len that the sample reads: every line when the row has fewer.
GS_HD int64_t pre_lines(int64_t len) {
  const int64_t nl = len / 16, ns = (int64_t)kPreWG * kPreLines;
  return nl < ns ? nl : ns;
}
// Refinement over candidates: at least kCandShare keys per chunk and at most kCandGroups chunks.
constexpr int64_t kCandShare = 1 << 13;
constexpr int64_t kCandGroups = 128;
// keys a lane buffers in LDS before its wave flushes (an odd stride keeps the lanes on different
// banks); sized so that the statistics workgroup stays within a quarter of the LDS (four resident
// per compute unit)
constexpr int kCandLane = 7;
// Candidate capacity per row a full workspace provides.
GS_HD int64_t cand_cap_full(int64_t d) {
  if (d < kCandMinRow) return 0;
  int64_t c = d / 16;
  if (c < ((int64_t)1 << 20)) c = (int64_t)1 << 20;
  return (c < d ? c : d) & ~(int64_t)63;  // whole 256-byte blocks
}

// Histogram copies: row r's copy c of level 1 is h1 + (r * kC1 + c).
// cand_cap: candidate keys per row (the workspace ends with the candidate buffers, so a smaller
// capacity changes no other offset).
GS_HD Layout layout_of(int64_t rows, int64_t d, int64_t cand_cap) {
  Layout L;
  L.tiles = (d + kTileElems - 1) / kTileElems;
  size_t off = 256;  // header (reserved)
  L.ctl = off;
  off += align256((size_t)rows * sizeof(RowCtl));
  L.h1 = off;
  off += align256((size_t)rows * kC1 * sizeof(Hist1));
  L.scratch = off;
  off += (size_t)rows * sizeof(RowScratch);
  L.kc = off;
  off += align256((size_t)rows * 8 * sizeof(CountLine));
  L.status = off;
  off += align256((size_t)rows * (size_t)L.tiles * sizeof(uint64_t));
  // segmented calls: workgroup -> (row, block) of the histogram passes and (row, first tile) of the
  // sample pass, for the workgroups that hold coordinates only
  L.bmap = off;
  off += align256((size_t)rows * (size_t)((d + kMinChunk - 1) / kMinChunk) * sizeof(uint64_t));
  L.tmap = off;
  off += align256((size_t)rows * (size_t)L.tiles * sizeof(uint64_t));
  // variance-budget solver only
  L.h1q = off;
  off += align256((size_t)rows * kC1 * sizeof(H1Q));
  // candidate band
  L.pre = off;
  off += align256((size_t)rows * sizeof(PreHist));
  L.ccnt = off;  // per row: keys collected (reserved in the compact list)
  off += align256((size_t)rows * sizeof(CountLine));
  L.cand = off;  // per row: the compact candidate list, then the statistics workgroups' regions
  L.cand_cap = cand_cap;
  off += align256((size_t)rows * (size_t)cand_cap * 2 * sizeof(uint32_t));
  L.total = off;
  return L;
}

struct Args {
  const float* g;
  int64_t rows, d, ld;
  const double* rho_dev;  // per-row densities, or nullptr to use `rho`
  double rho;
  const uint64_t* seed_dev;
  uint64_t seed;
  int solver, T;
  char* ws;
  Layout lay;
  int nb;          // workgroups per row of the histogram passes
  int64_t chunk;   // elements per histogram workgroup (multiple of 4)
  int32_t* idx;    // compaction: every survivor; hybrid coding: Q_A, the capped survivors
  float* val;
  int64_t cap;
  int64_t* nnz;
  int32_t* code_b;  // hybrid coding: Q_B, index | sign << 31 of every other survivor
  int64_t cap_b;
  int64_t* nnz_b;
  float* inv_out;   // hybrid coding: fp32 1/lambda per row
  int8_t* q;        // hybrid coding: optional dense ternary vector, leading dimension ld
  double* lam_out;
  int64_t* k_out;
  uint32_t* flags_out;
  float* p;
  // segmented calls: row r is g[seg[r], seg[r + 1]) (device offsets), d the longest segment
  const int64_t* seg;
  int64_t seg_total;  // the host's last offset: no segment may end beyond it
  int64_t seg_elems;  // the host's total segment length
  int64_t seg_chunk;  // host: histogram-pass chunk chosen from the segment lengths
  int64_t seg_tiles;  // host: sample tiles that hold coordinates, over all segments
  int64_t seg_blocks; // histogram-pass workgroups (the grid), from the host offsets
  int64_t seg_rest;   // those of them past their segment's first
  int64_t seg_wgs;    // sample-pass workgroups (the grid), from the host offsets
  int seg_k;          // tiles per sample workgroup
  int seg_align;      // the host's offsets are multiples of 4 (and g 16-byte aligned): the device's must be too
  size_t ws_bytes;    // the workspace's size (the candidate buffers take what the rest leaves)
  int64_t cand_region;  // candidate keys per statistics workgroup (cand_cap / nb, a multiple of 64)
  int help_step;        // histogram chunks past a row's first per helper of the solver
  int helpers;          // helpers per row of a strided batch
};

// Start and length of row r: row r of a strided batch (offset r * ld, length d), or segment r of a
// segmented call. A segment whose device offsets break the bounds the host checked (order, end,
// length, alignment where the host's offsets are aligned) reads as empty and returns false.
__device__ __forceinline__ bool row_span(const Args& a, int64_t r, int64_t& base, int64_t& len) {
  if (!a.seg) {
    base = r * a.ld;
    len = a.d;
    return true;
  }
  const int64_t b = a.seg[r], e = a.seg[r + 1];
  const bool ok = b >= 0 && e >= b && e <= a.seg_total && e - b <= a.d && (!a.seg_align || (b & 3) == 0);
  base = ok ? b : 0;
  len = ok ? e - b : 0;
  return ok;
}

// Segmented calls: the word k_init leaves in the workspace header, 1 when the workgroup maps built
// from the device offsets have exactly the host's shape (the launched grids), 2 when they do not
// (every segment is then flagged GSPAR_FLAG_BADSEG and skipped).
__device__ __forceinline__ uint32_t* segok_of(const Args& a) { return reinterpret_cast<uint32_t*>(a.ws); }

__device__ __forceinline__ RowCtl* ctl_of(const Args& a, int64_t r) {
  return reinterpret_cast<RowCtl*>(a.ws + a.lay.ctl) + r;
}
__device__ __forceinline__ Hist1* h1_of(const Args& a, int64_t r, int c = 0) {
  return reinterpret_cast<Hist1*>(a.ws + a.lay.h1) + r * kC1 + c;
}
__device__ __forceinline__ RowScratch* scratch_of(const Args& a, int64_t r) {
  return reinterpret_cast<RowScratch*>(a.ws + a.lay.scratch) + r;
}
__device__ __forceinline__ H1Q* h1q_of(const Args& a, int64_t r, int c = 0) {
  return reinterpret_cast<H1Q*>(a.ws + a.lay.h1q) + r * kC1 + c;
}
__device__ __forceinline__ CountLine* kc_of(const Args& a, int64_t r) {
  return reinterpret_cast<CountLine*>(a.ws + a.lay.kc) + r * 8;
}
__device__ __forceinline__ uint64_t* status_of(const Args& a) {
  return reinterpret_cast<uint64_t*>(a.ws + a.lay.status);
}
__device__ __forceinline__ PreHist* pre_of(const Args& a, int64_t r) {
  return reinterpret_cast<PreHist*>(a.ws + a.lay.pre) + r;
}
// Candidates of row r: the compact list (cand_cap keys), then the staging regions, where statistics
// workgroup b collects into keys [b * cand_region, (b + 1) * cand_region) before moving them to
// the list; the row's count line holds the keys reserved in the list.
__device__ __forceinline__ CountLine* ccnt_of(const Args& a, int64_t r) {
  return reinterpret_cast<CountLine*>(a.ws + a.lay.ccnt) + r;
}
__device__ __forceinline__ uint32_t* cand_of(const Args& a, int64_t r) {
  return reinterpret_cast<uint32_t*>(a.ws + a.lay.cand) + r * a.lay.cand_cap * 2;
}
__device__ __forceinline__ uint32_t* creg_of(const Args& a, int64_t r) { return cand_of(a, r) + a.lay.cand_cap; }



// Orders the LDS accesses of a wave's lanes for the compiler (the wave issues them in order as it is):
// what a lane reads or writes before, it does before any lane's accesses after. No instruction.
__device__ __forceinline__ void wave_sync() {
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#endif
  __builtin_amdgcn_wave_barrier();
}
// LDS bytes reused as 16-bit words.
typedef uint16_t __attribute__((may_alias)) gs_u16;

// Streaming accesses: g is read once per pass and the outputs are written once, so those loads (the
// solver's list requests apart, where the hint makes 16 rows of 2^20 under the variance budget faster,
// 130 us a call against 135, and 300 rows of 200,001 and the probabilities of 2^26 coordinates slower,
// 209 against 203 and 339 against 328),
// the probabilities' stores and the sampling pass's staged stores (whole runs of consecutive words)
// carry the non-temporal hint and do not displace what the caches keep (the level-1 copies,
// windows and status words). Stores that lanes make one word at a time to scattered places (the
// other emission paths, the hybrid coding's Q_A list, the candidate band) keep the default policy:
// there the hint made the hybrid coding's sampling pass a third slower at rho = 0.1. On 2^28
// coordinates the hint takes the statistics pass from about 213 to 192 microseconds per call.
//
// A row may start at any float (odd leading dimensions, segments, views): global memory takes
// 16-byte accesses at any multiple of 4 bytes, so the vector type below asks for no more and every
// row streams through the same loops. With a scalar-load copy of every loop for such rows, and the
// solver still in several launches, 5 rows of 300,007 in a packed matrix took 77 us a call against 70,
// one odd row of a few million coordinates whose solver refines 159 against 98 us; rows on 16-byte
// boundaries issue the same instructions.
#if defined(__HIP_DEVICE_COMPILE__)
typedef float gs_f4v __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ float4 load_vec(const float* p) {
  const gs_f4v v = *reinterpret_cast<const gs_f4v*>(p);
  return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ float4 load_stream(const float* p) {
  const gs_f4v v = __builtin_nontemporal_load(reinterpret_cast<const gs_f4v*>(p));
  return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void store_stream(float* p, float4 x) {
  const gs_f4v v = {x.x, x.y, x.z, x.w};
  __builtin_nontemporal_store(v, reinterpret_cast<gs_f4v*>(p));
}
#define GS_STORE_STREAM(ptr, v) __builtin_nontemporal_store((v), (ptr))
#else
GS_HD float4 load_vec(const float* p) {
  float4 x;
  memcpy(&x, p, sizeof(x));
  return x;
}
GS_HD float4 load_stream(const float* p) { return load_vec(p); }
GS_HD void store_stream(float* p, float4 x) { memcpy(p, &x, sizeof(x)); }
#define GS_STORE_STREAM(ptr, v) (*(ptr) = (v))
#endif

// Four consecutive coordinates 4q..4q+3 of a row; entries at or beyond `end` read as 0 and are
// flagged invalid in the returned mask (bit c set = coordinate 4q+c exists).
__device__ __forceinline__ uint32_t load4(const float* __restrict__ row, int64_t q, int64_t end, float v[4]) {
  const int64_t i = 4 * q;
  if (i + 3 < end) {
    const float4 x = load_vec(row + i);
    v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
    return 0xF;
  }
  uint32_t m = 0;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    bool ok = i + c < end;
    v[c] = ok ? row[i + c] : 0.0f;
    m |= (uint32_t)ok << c;
  }
  return m;
}


// Visits the coordinates [beg, end) of one row (beg a multiple of 4) with the NT threads of a
// workgroup, calling f(q, v, m) for each float4 group q (m: bit c set when coordinate 4q+c exists).
// Blocks of U groups per thread are loaded unconditionally, all issued before any group is processed,
// so U loads per thread stay in flight; the last block clamps its addresses to the last whole group
// and masks the values, and a trailing partial group is loaded by one thread with scalar loads and
// visited by the whole first wave. No memory access sits under a divergent branch, which would make
// the compiler wait for every outstanding load. Every call of f is made by whole waves, so f may use
// cross-lane operations.
template <int U, int NT, typename F>
__device__ __forceinline__ void stream_groups(const float* __restrict__ row, int64_t beg, int64_t end, F&& f) {
  const int64_t qfull = end / 4;  // groups [beg/4, qfull) lie entirely inside [beg, end)
  int64_t qb = beg / 4;
  for (; qb + (int64_t)U * NT <= qfull; qb += (int64_t)U * NT) {
    float4 x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) x[u] = load_stream(row + 4 * (qb + threadIdx.x + u * NT));
    __builtin_amdgcn_sched_barrier(0);  // keep every load of the block ahead of the first use
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float v[4] = {x[u].x, x[u].y, x[u].z, x[u].w};
      f(qb + threadIdx.x + u * NT, v, 0xFu);
    }
  }
  if (qb < qfull) {
    float4 x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t q = qb + threadIdx.x + u * NT;
      x[u] = load_vec(row + 4 * (q < qfull ? q : qfull - 1));
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t q = qb + threadIdx.x + u * NT;
      const bool ok = q < qfull;
      float v[4] = {ok ? x[u].x : 0.0f, ok ? x[u].y : 0.0f, ok ? x[u].z : 0.0f, ok ? x[u].w : 0.0f};
      f(q, v, ok ? 0xFu : 0u);
    }
  }
  if (4 * qfull < end && threadIdx.x < 64) {
    // the last, partial group: visited by the whole first wave (its other lanes see no
    // coordinates), so a visitor may use cross-lane operations
    float v[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    uint32_t m = 0;
    if (threadIdx.x == 0) m = load4(row, qfull, end, v);
    f(qfull, v, m);
  }
}

// The same in blocks of U groups per thread, f(x) for each (coordinates outside [beg, end) read as 0),
// for visitors with work to do once per block.
template <int U, int NT, typename F>
__device__ __forceinline__ void stream_blocks(const float* __restrict__ row, int64_t beg, int64_t end, F&& f) {
  const int64_t qfull = end / 4;
  int64_t qb = beg / 4;
  float4 x[U];
  for (; qb < qfull; qb += (int64_t)U * NT) {
    const bool whole = qb + (int64_t)U * NT <= qfull;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t q = qb + threadIdx.x + u * NT;
      x[u] = load_vec(row + 4 * (q < qfull ? q : qfull - 1));
    }
    __builtin_amdgcn_sched_barrier(0);
    if (!whole) {
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (qb + threadIdx.x + u * NT >= qfull) x[u] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    }
    f(x);
  }
  if (4 * qfull < end && threadIdx.x < 64) {
#pragma unroll
    for (int u = 0; u < U; ++u) x[u] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    float v[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (threadIdx.x == 0) load4(row, qfull, end, v);
    x[0] = make_float4(v[0], v[1], v[2], v[3]);
    f(x);
  }
}

// Helpers of the histogram passes and the solver are force-inlined, so LDS and global pointers keep
// their address spaces and no call frames or scratch are needed.
#define GS_DI __device__ __attribute__((always_inline)) inline

// LDS of the statistics pass: per binade and lane class, (count << 44) | significand sum and the
// maximum key. Counts stay below 2^20 per workgroup, so significand sums stay below 2^44.
struct StatsLds {
  unsigned long long pk[kB1 * kLaneCopies];
  uint32_t mx[kB1 * kLaneCopies];
};
// with the squared significands of the variance-budget solver (split at bit 24, see H1Q)
template <bool SQ>
struct StatsLdsT : StatsLds {};
template <>
struct StatsLdsT<true> : StatsLds {
  unsigned long long qh[kB1 * kLaneCopies];
  unsigned long long ql[kB1 * kLaneCopies];
};
// popcount(m & bits of the lanes below this one)
__device__ __forceinline__ uint32_t lanes_below(unsigned long long m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}
// Exclusive prefix over the lanes of a wave of x in [0, 2^B) from B ballots; `total` receives the
// wave's sum.
template <int B>
__device__ __forceinline__ uint32_t wave_prefix_bits(uint32_t x, uint32_t& total) {
  uint32_t pre = 0;
  total = 0;
#pragma unroll
  for (int b = 0; b < B; ++b) {
    const unsigned long long m = __ballot((x >> b) & 1);
    pre += lanes_below(m) << b;
    total += (uint32_t)__popcll(m) << b;
  }
  return pre;
}

// ------------------------------------------------------------------------------------------
// The solver: one kernel after the statistics pass, k_solve, with a leading workgroup per row
// (workgroups 0 .. rows - 1) and helpers for the rows of more than one histogram chunk.
//
// What bounds it is latency: a row needs its 256 binades, then (only if a capped threshold falls
// inside a binade that holds several keys) the keys of that binade, which may take a pass over the
// row. The leader decides everything; a pass over the row (or over its candidates) is a request in
// the row's control block that every workgroup of the row takes chunks of. One launch does it all:
// a row that needs no pass costs one short kernel (8-9 us), where a launch for every possible
// pass and solve cost 23 us (11 us for the first solve, the rest idle kernels). By this change alone a
// call on 65,536 coordinates went from 38.9 us to 26.8, the 54 layers of a residual network from 96.6
// to 73.7, 5 rows of 300,007 whose solver lists a binade from 70 to 44, and 2^28 coordinates from 483
// to 457 (exact, rho = 0.01) and from 571 to 539 (greedy, rho = 0.1).
//
// Waiting: a chunk is taken with an atomic on its own word by its helper, or by the leader once it
// has done its own, so a chunk is only ever held by a running workgroup and the leader waits only
// for chunks that were taken: no wait depends on another workgroup being scheduled. Helpers are
// optional (the leader alone would take every chunk); one that finds no request for long enough
// leaves. About kSolveHelpers of them are launched at most, as many as are resident at once, and one
// that is done with its own chunk takes others: with helpers bound to one chunk each, the 1,025 chunks
// of a row of 2^30 coordinates were left to the leader where they found no helper resident (15.4 ms a
// call under the variance budget and 99 ms where the greedy solver counts over an unaligned row, against
// 3.0 and 3.5), and so were those of calls on several streams, whose helpers held each other off the
// compute units (one row of 2^24, exact, on four streams: 1,033 us a call against 74). Hand-offs use
// agent-scope atomics for the data itself as well as for the words that announce it, each side waiting
// for its own accesses to complete (s_waitcnt) before it announces them, so no cache write-back or
// invalidation is needed. Every word that all chunks would touch is avoided: atomics on one address take
// 10-30 ns each (counting a 2^28 row's candidates through one counter per wave took 150 us a request).
//
// Exact and variance solver: descend from binades (2^23 keys) to windows of 512 bins, of 2^14, then
// 2^5, then single keys. At each level the highest bin whose maximum passes the criterion (b1) and
// the lowest occupied bin above it (b2): the answer is b1's maximum unless b2 holds two or more keys
// that could still pass, in which case b2 is the next window. A range of at most kListCap keys is
// collected into a list once and every further level is binned from it by the leader.
// ------------------------------------------------------------------------------------------
enum : uint32_t { kReqWindow = 1, kReqList = 2, kReqCount = 3 };
constexpr uint32_t kReqDone = 255;      // request number: the row is solved
constexpr int kHelperPolls = 1 << 15;   // some 20 ms without a request
// Helpers of a call: the solver's workgroups that are resident at once (two on each of 256 compute
// units). Calls whose chunks are shorter than kMaxChunk have fewer chunks than this, and a helper for
// each. With 256 of them calls that list a binade take 5 to 15 per cent longer when alone (16 x 2^20,
// greedy, rho = 0.1: 80 us against 72) and less when several streams share the chip (on four streams 49
// against 58). (A build may lower it to give a helper several chunks on small inputs.)
#ifndef GSPAR_SOLVE_HELPERS
#define GSPAR_SOLVE_HELPERS 512
#endif
constexpr int64_t kSolveHelpers = GSPAR_SOLVE_HELPERS;
constexpr int kListBatch = 8;           // listed keys in flight per thread of the leader
constexpr int kPassBuf = 4096;          // listed keys a workgroup gathers in LDS before it appends them

template <class T>
GS_DI T ld_agent(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class T>
GS_DI void st_agent(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// A value every lane holds equally, moved to scalar registers.
template <class T>
GS_DI T uni(T v) {
#if defined(__HIP_DEVICE_COMPILE__)
  static_assert(sizeof(T) % 4 == 0, "whole registers");
  uint32_t w[sizeof(T) / 4];
  memcpy(w, &v, sizeof(T));
#pragma unroll
  for (int i = 0; i < (int)(sizeof(T) / 4); ++i) w[i] = __builtin_amdgcn_readfirstlane(w[i]);
  memcpy(&v, w, sizeof(T));
#endif
  return v;
}
// Every access of this wave so far has completed. (The fence is for the compiler, which may otherwise
// take the wait to have nothing to do with memory: no instruction.)
GS_DI void wait_own() {
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#endif
  __builtin_amdgcn_s_waitcnt(0);
}

// One request. The leader announces it as one word, so that a helper needs no second look:
// bits 0-31 the range's first key (kReqCount: the query key), 32-39 its number, 40-41 its kind, 42
// set when the chunks are of the row's candidates, 43-44 the range: a binade, 2^14 or 2^5 keys.
struct Pass {
  uint32_t key, num, kind, from, shift;
};
GS_DI uint64_t pass_word(const Pass& P) {
  const uint32_t lev = P.shift == 14 ? 0u : (P.shift == 5 ? 1u : 2u);
  return ((uint64_t)(P.num | (P.kind << 8) | (P.from << 10) | (lev << 11)) << 32) | P.key;
}
GS_DI Pass pass_of(uint64_t w) {
  const uint32_t h = (uint32_t)(w >> 32), lev = h >> 11;
  Pass P;
  P.key = (uint32_t)w;
  P.num = h & 0xFFu;
  P.kind = (h >> 8) & 3u;
  P.from = (h >> 10) & 1u;
  P.shift = lev == 0 ? 14u : (lev == 1 ? 5u : 0u);
  return P;
}
// The chunks of the row, or of its candidates: equal shares of whole groups of 4, at least kCandShare
// keys each, at most kCandGroups shares. n: the source's length.
GS_DI void pass_chunks(const Args& a, uint32_t from, int64_t n, int64_t& share, uint32_t& chunks) {
  share = a.chunk;
  if (from) {
    const int64_t groups = min((int64_t)a.nb, kCandGroups);
    share = max(kCandShare, (((n + groups - 1) / groups) + 3) & ~(int64_t)3);
  }
  chunks = (uint32_t)((n + share - 1) / share);
}

// LDS of a window binned by one workgroup: kWC copies by lane. pk: (count << 44) | sum of offsets
// within the bin (fewer than 2^20 keys a time, offsets below 2^14).
template <bool VAR>
struct WinLds {
  unsigned long long pk[kWB * kWC];
  unsigned long long s2[VAR ? kWB * kWC : 1];
  uint32_t mx[kWB * kWC];
};
// A bin of the level under examination, broadcast by the thread that owns it.
struct BinOut {
  uint64_t part;   // significand sum of the keys of binade E up to and including the bin
  uint64_t ph, pl; // and of their squares (bits above 24, low part)
  uint64_t sig, sh, sl;  // the bin's own sums
  uint32_t below;  // keys of the row up to and including the bin
  uint32_t cnt, mx, state;
};
template <bool VAR>
struct SolveLds {
  uint32_t cnt[kB1];   // level 1: per binade the count, significand sum, maximum key
  uint64_t sig[kB1];
  uint32_t mx[kB1];
  uint32_t pc[kB1];    // count of the keys of the binades up to and including this one
  double pw[kB1];      // about their sum
  uint64_t qh[VAR ? kB1 : 1];
  uint64_t ql[VAR ? kB1 : 1];
  double pq[VAR ? kB1 : 1];
  unsigned long long dig[kDigSq];
  int hi[2][kNT / 64];
  uint32_t rc[kNT / 64];
  uint64_t rs[kNT / 64], rh[kNT / 64], rl[kNT / 64];
  double rw[kNT / 64], rq[kNT / 64];
  BinOut bin[2], ans;  // the bins b1 and b2 as their owners see them; the answer so far
  uint64_t word;       // a helper's next request (0: leave)
  uint32_t cmd;        // whether the chunk at hand was taken by this workgroup
  uint32_t err;        // kFlagInternal when a shift of the leader's exact sums lay outside its range
  uint32_t next;       // a helper's next chunk (0: none)
  uint32_t nbuf, base;  // keys of the chunk at hand that belong in the list, and their place there
  uint32_t keys[kPassBuf];  // the leader's first listed keys
  union {
    WinLds<VAR> win;
    uint32_t buf[kPassBuf];
  };
};
static_assert(kPassBuf == kListBatch * kNT, "one batch fills the leader's keys");

// Block-wide: the highest (HIGH) or lowest thread with pred; -1 or kNT when there is none. Two
// result rows used in turn, so one barrier per search.
template <bool HIGH, class S>
GS_DI int block_find(S& s, uint32_t& turn, bool pred) {
  const unsigned long long m = __ballot(pred);
  const int wv = threadIdx.x >> 6;
  turn ^= 1u;
  if ((threadIdx.x & 63) == 0)
    s.hi[turn][wv] = m ? wv * 64 + (HIGH ? 63 - __builtin_clzll(m) : __builtin_ctzll(m)) : (HIGH ? -1 : kNT);
  __syncthreads();
  int r = s.hi[turn][0];
#pragma unroll
  for (int i = 1; i < kNT / 64; ++i) r = HIGH ? max(r, s.hi[turn][i]) : min(r, s.hi[turn][i]);
  return uni(r);
}

template <class T>
GS_DI T wave_incl(T x, int lane) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const T y = __shfl_up(x, o);
    if (lane >= o) x += y;
  }
  return x;
}

// The exact sum of every magnitude of the binades below E and of the keys of binade E whose
// significands add up to `part`, rounded once. Every thread calls it and receives the sum.
template <class S>
GS_DI double exact_sum(S& s, int E, uint64_t part) {
  const int t = threadIdx.x;
  if (t < kDig) s.dig[t] = 0;
  __syncthreads();
  const uint64_t v = t < E && t < kB1 ? s.sig[t] : (t == E ? part : 0ull);
  if (v) {
    int at;
    uint64_t x[3];
    if (dig_split(v, binade_shift(t), 255, at, x)) s.err = kFlagInternal;
#pragma unroll
    for (int i = 0; i < 3; ++i) atomicAdd(&s.dig[at + i], (unsigned long long)x[i]);
  }
  __syncthreads();
  const double r = uni(dig_round<kDig>(s.dig, -149));
  __syncthreads();
  return r;
}
// The same for the squares; `ph`, `pl` as in H1Q.
template <class S>
GS_DI double exact_sum_sq(S& s, int E, uint64_t ph, uint64_t pl) {
  const int t = threadIdx.x;
  if (t < kDigSq) s.dig[t] = 0;
  __syncthreads();
  const bool own = t < E && t < kB1;
  const uint64_t vh = own ? s.qh[t] : (t == E ? ph : 0ull), vl = own ? s.ql[t] : (t == E ? pl : 0ull);
  if (vh | vl) {
    int at;
    uint64_t x[3];
    uint32_t err = dig_split(vh, 2 * binade_shift(t) + 24, 2 * 255 + 24, at, x);
#pragma unroll
    for (int i = 0; i < 3; ++i) atomicAdd(&s.dig[at + i], (unsigned long long)x[i]);
    err |= dig_split(vl, 2 * binade_shift(t), 2 * 255, at, x);
#pragma unroll
    for (int i = 0; i < 3; ++i) atomicAdd(&s.dig[at + i], (unsigned long long)x[i]);
    if (err) s.err = err;
  }
  __syncthreads();
  const double r = uni(dig_round<kDigSq>(s.dig, -298));
  __syncthreads();
  return r;
}

// Works on chunk c of a request and puts the results into the row's scratch, if the chunk is this
// workgroup's: it is taken (with an atomic whose answer is needed only at the end) unless `own`
// says that it is already. Returns the request's chunks. Every thread of the workgroup calls it.
template <bool VAR>
GS_DI uint32_t pass_chunk(const Args& a, SolveLds<VAR>& s, RowCtl* ctl, RowScratch* sc, int64_t row, int64_t base,
                      int64_t len, uint32_t c, const Pass& P, bool own) {
  const int64_t n = P.from ? (int64_t)ccnt_of(a, row)->v : len;
  int64_t share;
  uint32_t chunks;
  pass_chunks(a, P.from, n, share, chunks);
  if (c >= chunks) return chunks;
  uint32_t taken = 0;
  if (threadIdx.x == 0 && !own) taken = atomicMax(&sc->chunk[c].taken, P.num);
  const uint32_t lc = threadIdx.x & (kWC - 1);
  const float* src = P.from ? reinterpret_cast<const float*>(cand_of(a, row)) : a.g + base;
  const int64_t beg = (int64_t)c * share, end = min(n, beg + share);
  // the range; for kReqCount the keys of the query key's binade from it on
  const uint32_t lo = P.kind == kReqCount ? (P.key & 0x7F800000u) : P.key;
  const uint32_t span = P.shift ? (uint32_t)kWB << P.shift : 32u;
  auto claim = [&]() {
    if (threadIdx.x == 0) s.cmd = own || taken < P.num ? 1u : 0u;
    __syncthreads();
    return uni(s.cmd) != 0;
  };
  if (P.kind == kReqWindow) {
    for (int i = threadIdx.x; i < kWB * kWC; i += kNT) {
      s.win.pk[i] = 0;
      s.win.mx[i] = 0;
      if constexpr (VAR) s.win.s2[i] = 0;
    }
    __syncthreads();
    const uint32_t omask = (1u << P.shift) - 1u;
    stream_groups<4, kNT>(src, beg, end, [&](int64_t, const float v[4], uint32_t) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t key = key_of(v[k]), rel = key - lo;
        if (key != 0 && rel < span) {
          const uint32_t i = (rel >> P.shift) * kWC + lc, r = rel & omask;
          atomicAdd(&s.win.pk[i], (1ull << 44) | (unsigned long long)r);
          if constexpr (VAR) atomicAdd(&s.win.s2[i], (unsigned long long)r * r);
          atomicMax(&s.win.mx[i], rel);
        }
      }
    });
    if (!claim()) return chunks;
    const int b = threadIdx.x;
    uint64_t cnt = 0, sr = 0, s2 = 0;
    uint32_t mx = 0;
#pragma unroll
    for (int j = 0; j < kWC; ++j) {
      const uint64_t p = s.win.pk[b * kWC + j];
      cnt += p >> 44;
      sr += p & ((1ull << 44) - 1);
      mx = max(mx, s.win.mx[b * kWC + j]);
      if constexpr (VAR) s2 += s.win.s2[b * kWC + j];
    }
    if (cnt) {
      WinBins* w = &sc->win[c % kWC];
      atomicAdd(&w->cnt[b], (uint32_t)cnt);
      if (sr) atomicAdd((unsigned long long*)&w->sr[b], (unsigned long long)sr);
      if constexpr (VAR) {
        if (s2) atomicAdd((unsigned long long*)&w->s2[b], (unsigned long long)s2);
      }
      atomicMax(&w->mx[b], mx);
    }
  } else if (P.kind == kReqList) {
    if (threadIdx.x == 0) s.nbuf = 0;
    __syncthreads();
    // the wave's keys of a block of groups: one reservation for all of them, in LDS while there is room
    auto gather = [&](const auto& x) {
      constexpr int U = (int)(sizeof(x) / sizeof(x[0]));
      static_assert(4 * U < 32, "a 5-bit count per thread");
      uint32_t hit = 0;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const float v[4] = {x[u].x, x[u].y, x[u].z, x[u].w};
#pragma unroll
        for (int k = 0; k < 4; ++k) hit |= (uint32_t)(key_of(v[k]) != 0 && key_of(v[k]) - lo < span) << (4 * u + k);
      }
      if (!__ballot(hit != 0)) return;
      uint32_t tot;
      uint32_t at = wave_prefix_bits<5>((uint32_t)__popc(hit), tot), b = 0;
      if ((threadIdx.x & 63) == 0) b = atomicAdd(&s.nbuf, tot);
      at += (uint32_t)__shfl((int)b, 0);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const float v[4] = {x[u].x, x[u].y, x[u].z, x[u].w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          if ((hit >> (4 * u + k)) & 1) {
            if (at < (uint32_t)kPassBuf) s.buf[at] = key_of(v[k]);
            ++at;
          }
        }
      }
    };
    stream_blocks<4, kNT>(src, beg, end, gather);
    if (!claim()) return chunks;
    const uint32_t m = s.nbuf;
    if (threadIdx.x == 0 && m) s.base = atomicAdd(&ctl->lcount, m);
    __syncthreads();
    const uint32_t to = s.base;
    if (m <= (uint32_t)kPassBuf) {
      for (uint32_t i = threadIdx.x; i < m; i += kNT)
        if (to + i < (uint32_t)kListMax) st_agent(&sc->list[to + i], s.buf[i]);
    } else {
      // more than the buffer holds: read the chunk again, straight to the list
      if (threadIdx.x == 0) s.nbuf = to;
      __syncthreads();
      stream_groups<4, kNT>(src, beg, end, [&](int64_t, const float v[4], uint32_t) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const uint32_t key = key_of(v[k]);
          if (key != 0 && key - lo < span) {
            const uint32_t i = atomicAdd(&s.nbuf, 1u);
            if (i < (uint32_t)kListMax) st_agent(&sc->list[i], key);
          }
        }
      });
    }
  } else {
    uint32_t qc = 0;
    uint64_t qs = 0;
    stream_groups<4, kNT>(src, beg, end, [&](int64_t, const float v[4], uint32_t) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t key = key_of(v[k]);
        if (key >= P.key && key - lo < span) {
          ++qc;
          qs += key_sig(key);
        }
      }
    });
    for (int o = 32; o > 0; o >>= 1) {
      qc += __shfl_xor(qc, o);
      qs += __shfl_xor(qs, o);
    }
    if ((threadIdx.x & 63) == 0) {
      s.rc[threadIdx.x >> 6] = qc;
      s.rs[threadIdx.x >> 6] = qs;
    }
    if (!claim()) return chunks;
    if (threadIdx.x == 0) {
      for (int i = 1; i < kNT / 64; ++i) {
        qc += s.rc[i];
        qs += s.rs[i];
      }
      st_agent(&sc->chunk[c].qcnt, qc);
      st_agent(&sc->chunk[c].qsig, qs);
    }
  }
  wait_own();
  __syncthreads();  // every wave's results have landed, and the LDS may be reused
  if (threadIdx.x == 0) st_agent(&sc->chunk[c].done, P.num);
  return chunks;
}

// Helper h (from 1) of `helpers`: works on chunk h of each of the row's requests and, where no new
// request follows within kLookPolls, on chunks that nobody has taken by then, until the row is solved. It
// looks among those that differ from h by a multiple of `mod`, the helpers' number over 8 to 16 (a
// power of two, at most 64), with one load per lane, and takes the one at its own place among the
// helpers that share them; so the first eighth of the helpers covers every chunk where the others found
// no place, be it that the row has more chunks than helpers fit or that other streams' kernels hold the
// compute units. (Looking at once took chunks from helpers that were about to begin: a call whose solver
// counts twice over 2^22 coordinates took 46 us against 43.)
constexpr int kLookPolls = 2;  // some 1.2 us
template <bool VAR>
GS_DI void help_row(const Args& a, SolveLds<VAR>& s, RowCtl* ctl, RowScratch* sc, int64_t row, int64_t base,
                    int64_t len, uint32_t h, uint32_t helpers) {
  uint32_t seen = 0;  // thread 0: the last request looked at
  const uint32_t lg = 31u - (uint32_t)__builtin_clz(helpers), mod = 1u << (lg < 3 ? 0u : min(lg - 3u, 6u));
  Pass P{0, 0, 0, 0, 0};
  uint32_t chunks = 0;       // of the request P
  int polls = kHelperPolls;  // before it looks for a chunk (fewer than kHelperPolls) or leaves
  while (true) {
    if (threadIdx.x == 0) {
      uint64_t word = 0;
      for (int i = 0; i < polls; ++i) {
        word = ld_agent(&ctl->req);
        const uint32_t num = (uint32_t)(word >> 32) & 0xFFu;
        if (num != seen) {
          seen = num;
          break;
        }
        word = 0;
        __builtin_amdgcn_s_sleep(8);
      }
      s.word = word;
    }
    __syncthreads();
    const uint64_t word = uni(s.word);
    uint32_t c = h;
    if (word) {
      P = pass_of(word);
      if (P.num == kReqDone) return;
    } else if (polls == kHelperPolls) {
      return;
    } else {
      if (threadIdx.x < 64) {
        uint32_t next = 0;  // 0: nothing left (chunk 0 is the leader's)
        uint32_t b = h & (mod - 1u);
        while (b < chunks) {
          const uint32_t at = b + mod * threadIdx.x;
          unsigned long long m = __ballot(at != 0 && at < chunks && ld_agent(&sc->chunk[at].taken) < P.num);
          if (!m) {
            b += 64u * mod;
            continue;
          }
          for (uint32_t skip = (h / mod) % (uint32_t)__popcll(m); skip; --skip) m &= m - 1ull;
          next = b + mod * (uint32_t)__builtin_ctzll(m);
          uint32_t was = 0;
          if (threadIdx.x == 0) was = atomicMax(&sc->chunk[next].taken, P.num);
          if ((uint32_t)__shfl((int)was, 0) < P.num) break;  // else somebody took it in between: look again
          next = 0;
        }
        if (threadIdx.x == 0) s.next = next;
      }
      __syncthreads();
      c = uni(s.next);
      if (c == 0) {
        polls = kHelperPolls;
        continue;
      }
    }
    chunks = pass_chunk<VAR>(a, s, ctl, sc, row, base, len, c, P, word == 0);
    polls = word ? kLookPolls : 0;
    __syncthreads();
  }
}

// The leader's running state of a row.
struct Lead {
  uint32_t req = 0;      // requests made
  uint32_t turn = 0;
  bool banded = false;   // the candidate band is complete
  uint32_t blo = 0, bhi = 0;
  uint64_t cand_n = 0;
  uint32_t from = 0;     // source of the last request
  uint32_t chunks = 0;   // and its chunks
  uint32_t llo = 0, lspan = 0, ln = 0;  // the listed range's first key, whether there is one, its number of keys
};

// Makes a request, works on it and waits until all of it is done. `key`: the range's first key, for
// kReqCount the query key; `n`: the range's number of keys. The range lies in one binade.
template <bool VAR>
GS_DI void request(const Args& a, SolveLds<VAR>& s, RowCtl* ctl, RowScratch* sc, int64_t row, int64_t base,
                   int64_t len, Lead& L, uint32_t kind, uint32_t key, uint32_t shift, uint32_t n) {
  const uint32_t e = key >> 23;
  L.from = L.banded && (e << 23) >= L.blo && ((e + 1) << 23) <= L.bhi ? 1u : 0u;
  ++L.req;
  const Pass P{key, L.req, kind, L.from, shift};
  int64_t share;
  uint32_t chunks;
  pass_chunks(a, P.from, P.from ? (int64_t)L.cand_n : len, share, chunks);
  L.chunks = chunks;
  if (L.req == 1)
    for (uint32_t c = threadIdx.x; c < (uint32_t)a.nb && c < (uint32_t)kMaxChunks; c += kNT) {
      st_agent(&sc->chunk[c].taken, 0u);
      st_agent(&sc->chunk[c].done, 0u);
    }
  if (kind == kReqWindow) {
    uint64_t* w = reinterpret_cast<uint64_t*>(sc->win);
    for (int i = threadIdx.x; i < (int)(sizeof(sc->win) / 8); i += kNT) st_agent(&w[i], (uint64_t)0);
  }
  // (the list's counter starts at zero, and a row makes at most one list for each binade)
  if (kind == kReqList && L.lspan && threadIdx.x == 0) st_agent(&ctl->lcount, 0u);
  wait_own();
  __syncthreads();  // the scratch is clear: announce the request
  if (threadIdx.x == 0) st_agent(&ctl->req, pass_word(P));
  // its own chunk, chunks that no helper has taken by now (one copy of the code for both: the kernel's
  // instructions are mostly fetched once, from memory), then those that are still being worked on
  int f = 0;
  for (uint32_t c0 = 0; c0 < chunks; c0 += kNT) {
    const uint32_t c = c0 + threadIdx.x;
    while (true) {
      if (f != 0 || c0 != 0)
        f = block_find<false>(s, L.turn, c > 0 && c < chunks && ld_agent(&sc->chunk[c].taken) < P.num);
      if (f == kNT) break;
      pass_chunk<VAR>(a, s, ctl, sc, row, base, len, c0 + (uint32_t)f, P, c0 + (uint32_t)f == 0);
      __syncthreads();
      if (f == 0) f = kNT + 1;
    }
    while (block_find<false>(s, L.turn, c < chunks && ld_agent(&sc->chunk[c].done) != P.num) != kNT)
      __builtin_amdgcn_s_sleep(1);
  }
  if (kind == kReqList) {
    L.llo = key;
    L.lspan = 1;
    L.ln = n;
    // the first kPassBuf keys stay in LDS, each read by the thread that put it there
    uint32_t k[kListBatch];
#pragma unroll
    for (int j = 0; j < kListBatch; ++j) {
      const uint32_t i = threadIdx.x + j * kNT;
      k[j] = i < n ? ld_agent(&sc->list[i]) : 0u;
    }
#pragma unroll
    for (int j = 0; j < kListBatch; ++j) s.keys[threadIdx.x + j * kNT] = k[j];
  }
}

// Visits this thread's listed keys.
template <class S, class F>
GS_DI void each_listed(const S& s, const RowScratch* sc, const Lead& L, F&& f) {
  for (uint32_t i = threadIdx.x; i < min(L.ln, (uint32_t)kPassBuf); i += kNT) f(s.keys[i]);
  // the rest kListBatch at a time: one load after another took 0.4 us each, 7.6 us for 22,000 keys
  for (uint32_t b = kListBatch * kNT; b < L.ln; b += kListBatch * kNT) {
    uint32_t k[kListBatch];
#pragma unroll
    for (int j = 0; j < kListBatch; ++j) {
      const uint32_t i = b + threadIdx.x + j * kNT;
      k[j] = ld_agent(&sc->list[i < L.ln ? i : 0]);
      if (i >= L.ln) k[j] = 0;
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < kListBatch; ++j)
      if (k[j]) f(k[j]);
  }
}

// Count and significand sum of the keys >= t of t's binade.
GS_DI void count_above(const Args& a, SolveLds<false>& s, RowCtl* ctl, RowScratch* sc, int64_t row, int64_t base,
                       int64_t len, Lead& L, uint32_t t, uint64_t& qc, uint64_t& qs) {
  const uint32_t lo = (t >> 23) << 23, n = s.cnt[t >> 23];
  if (L.lspan == 0 || L.llo != lo) {
    const bool list = n <= kListCap;
    request<false>(a, s, ctl, sc, row, base, len, L, list ? kReqList : kReqCount, list ? lo : t, 14, n);
  }
  uint32_t c = 0;
  uint64_t g = 0;
  if (n > kListCap) {
    for (uint32_t i = threadIdx.x; i < L.chunks; i += kNT) {
      c += ld_agent(&sc->chunk[i].qcnt);
      g += ld_agent(&sc->chunk[i].qsig);
    }
  } else {
    each_listed(s, sc, L, [&](uint32_t key) {
      if (key >= t) {
        ++c;
        g += key_sig(key);
      }
    });
  }
  for (int o = 32; o > 0; o >>= 1) {
    c += __shfl_xor(c, o);
    g += __shfl_xor(g, o);
  }
  __syncthreads();
  if ((threadIdx.x & 63) == 0) {
    s.rc[threadIdx.x >> 6] = c;
    s.rs[threadIdx.x >> 6] = g;
  }
  __syncthreads();
  qc = 0;
  qs = 0;
  for (int i = 0; i < kNT / 64; ++i) {
    qc += s.rc[i];
    qs += s.rs[i];
  }
}

// Algorithm 2's criterion at a data value v, from K = #{a > v} and the rounded exact sums T1 (and,
// variance budget, T2) of the magnitudes up to v and of their squares. Density budget:
// (B - K) v <= T1; variance budget: v T1 <= eps A2 + T2 with every operation rounded on its own
// (the pragma keeps the compiler from fusing the product and the sum).
template <bool VAR>
GS_DI bool criterion(double B, double A2, uint64_t K, uint32_t vkey, double T1, double T2, double& lhs, double& rhs) {
#pragma clang fp contract(off)
  if constexpr (VAR) {
    lhs = key_value(vkey) * T1;
    const double eA = B * A2;
    rhs = eA + T2;
  } else {
    lhs = (B - (double)K) * key_value(vkey);
    rhs = T1;
  }
  return lhs <= rhs;
}

// The capped set of Proposition 1 is {p_i = 1}: the magnitudes above the criterion's value v
// (keys >= tcap = key(v) + 1) and, should fl(lambda * a) reach 1 below them (a tied run at v when
// the criterion holds with equality), those too. Both sets are {key >= t} for some t, so the union
// is the smaller threshold; every pass tests key >= the final tcap.
GS_DI uint32_t capped_threshold(double lam, uint32_t tcap) {
  const uint32_t t = cap_key(lam);
  return t < tcap ? t : tcap;
}

// The exact and the variance-budget solver (see above): lambda and the capped threshold of a row
// whose level-1 table is in LDS. Returns kFlagInternal when nothing passes (density budget: a broken
// invariant, the criterion holds at the smallest magnitude).
template <bool VAR>
GS_DI uint32_t solve_levels(const Args& a, SolveLds<VAR>& s, RowCtl* ctl, RowScratch* sc, int64_t row, int64_t base,
                            int64_t len, Lead& L, double B, uint64_t nnz, double A2, double& lam, uint32_t& tcap) {
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  // the level: bins of 2^shift keys from `lo` (level 1: thread t's bin is binade t), with `below` keys
  // of the row and the sums (bsig; bh, bl) of binade E below it
  int E = -1;
  uint32_t lo = 0, shift = 23, below = 0;
  uint64_t bsig = 0, bh = 0, bl = 0;
  bool have = false;  // an answer, unless a lower level gives a better one
  bool rounded = false;  // its sum T1 and the criterion's right-hand side are rounded
  int aE = 0;
  double T1 = 0.0, rhs = 0.0;
  while (true) {
    // this thread's bin: count, significand sum, largest key, square sums
    uint32_t cnt = 0, mx = 0;
    uint64_t sig = 0, qh = 0, ql = 0;
    if (E < 0) {
      if (t < kB1) {
        cnt = s.cnt[t];
        sig = s.sig[t];
        mx = s.mx[t];
        if constexpr (VAR) {
          qh = s.qh[t];
          ql = s.ql[t];
        }
      }
    } else {
      uint64_t sr = 0, s2 = 0;
      if (L.lspan) {
        __syncthreads();
        for (int i = t; i < kWB * kWC; i += kNT) {
          s.win.pk[i] = 0;
          s.win.mx[i] = 0;
          if constexpr (VAR) s.win.s2[i] = 0;
        }
        __syncthreads();
        const uint32_t lc = t & (kWC - 1), span = shift ? (uint32_t)kWB << shift : 32u, omask = (1u << shift) - 1u;
        each_listed(s, sc, L, [&](uint32_t key) {
          const uint32_t rel = key - lo;
          if (rel < span) {
            const uint32_t i = (rel >> shift) * kWC + lc, r = rel & omask;
            atomicAdd(&s.win.pk[i], (1ull << 44) | (unsigned long long)r);
            if constexpr (VAR) atomicAdd(&s.win.s2[i], (unsigned long long)r * r);
            atomicMax(&s.win.mx[i], rel);
          }
        });
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kWC; ++j) {
          const uint64_t p = s.win.pk[t * kWC + j];
          cnt += (uint32_t)(p >> 44);
          sr += p & ((1ull << 44) - 1);
          mx = max(mx, s.win.mx[t * kWC + j]);
          if constexpr (VAR) s2 += s.win.s2[t * kWC + j];
        }
      } else {
#pragma unroll
        for (int j = 0; j < kWC; ++j) {
          cnt += ld_agent(&sc->win[j].cnt[t]);
          sr += ld_agent(&sc->win[j].sr[t]);
          mx = max(mx, ld_agent(&sc->win[j].mx[t]));
          if constexpr (VAR) s2 += ld_agent(&sc->win[j].s2[t]);
        }
      }
      mx += lo;
      // the bin's keys are m0 + offset as significands
      const uint64_t m0 = key_sig(lo) + ((uint64_t)t << shift);
      sig = cnt * m0 + sr;
      if constexpr (VAR) {
        // sum (m0 + r)^2 = cnt m0^2 + 2 m0 sum r + sum r^2, below 2^79
        const unsigned __int128 q = (unsigned __int128)(m0 * m0) * cnt + (unsigned __int128)(2 * m0) * sr + s2;
        qh = (uint64_t)(q >> 24);
        ql = (uint64_t)q & 0xFFFFFFu;
      }
    }
    // inclusive prefixes over the bins: counts, exact significand sums, and the sums as doubles
    const int sh = binade_shift(E < 0 ? t : E);
    uint32_t pc = cnt;
    uint64_t ps = sig, ph = qh, pl = ql;
    double pw = cnt ? ldexp((double)sig, sh - 149) : 0.0, pq = 0.0;
    if constexpr (VAR) pq = cnt ? ldexp((double)qh * 0x1p24 + (double)ql, 2 * sh - 298) : 0.0;
#pragma unroll 1
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t yc = __shfl_up(pc, o);
      const uint64_t ys = __shfl_up(ps, o);
      const double yw = __shfl_up(pw, o);
      const bool in = lane >= o;
      pc += in ? yc : 0u;
      ps += in ? ys : 0ull;
      pw += in ? yw : 0.0;
      if constexpr (VAR) {
        const uint64_t yh = __shfl_up(ph, o), yl = __shfl_up(pl, o);
        const double yq = __shfl_up(pq, o);
        ph += in ? yh : 0ull;
        pl += in ? yl : 0ull;
        pq += in ? yq : 0.0;
      }
    }
    __syncthreads();
    if (lane == 63) {
      s.rc[wv] = pc;
      s.rs[wv] = ps;
      s.rw[wv] = pw;
      if constexpr (VAR) {
        s.rh[wv] = ph;
        s.rl[wv] = pl;
        s.rq[wv] = pq;
      }
    }
    __syncthreads();
    for (int i = 0; i < wv; ++i) {
      pc += s.rc[i];
      ps += s.rs[i];
      pw += s.rw[i];
      if constexpr (VAR) {
        ph += s.rh[i];
        pl += s.rl[i];
        pq += s.rq[i];
      }
    }
    if (E < 0) {
      if (t < kB1) {
        s.pw[t] = pw;
        if constexpr (VAR) s.pq[t] = pq;
      }
    } else {
      // the keys below the window: the binades below E and the lower part of E
      pw += (E > 0 ? s.pw[E - 1] : 0.0) + ldexp((double)bsig, sh - 149);
      if constexpr (VAR) pq += (E > 0 ? s.pq[E - 1] : 0.0) + ldexp((double)bh * 0x1p24 + (double)bl, 2 * sh - 298);
    }
    // what the criterion needs at this bin's maximum: keys up to the bin, sums of binade E up to it
    const uint32_t kb = below + pc;
    const uint64_t part = E < 0 ? sig : bsig + ps, parth = E < 0 ? qh : bh + ph, partl = E < 0 ? ql : bl + pl;
    // screen with the double sums (non-negative terms, each prefix within 2^-48 of its value): a margin
    // above 2^-44 decides as the exact evaluation would; the rest (2) is evaluated exactly
    uint32_t st = 0;
    if (cnt) {
      double lhs, about;
      criterion<VAR>(B, A2, nnz - kb, mx, pw, pq, lhs, about);
      const double tol = 0x1p-44 * (VAR ? lhs + about : about);
      st = lhs <= about - tol ? 1u : (lhs > about + tol ? 0u : 2u);
    }
    // b1: the highest bin whose maximum passes; b2: the lowest occupied bin above it (when no maximum
    // passes, the lowest occupied bin itself: the answer may be one of its smaller keys), refined
    // while it holds two or more keys. An answer's sums are rounded only when it may stand (one place
    // for all of it: the code runs once per level, and cold instructions cost more than these steps).
    BinOut o2;
    bool down;
    int b2;
    while (true) {
      const int b1 = block_find<true>(s, L.turn, st != 0);
      b2 = block_find<false>(s, L.turn, cnt != 0 && t > b1);
      if (t == b1 || t == b2) {
        BinOut& o = s.bin[t == b1 ? 0 : 1];
        o.part = part;
        o.ph = parth;
        o.pl = partl;
        o.sig = sig;
        o.sh = qh;
        o.sl = ql;
        o.below = kb;
        o.cnt = cnt;
        o.mx = mx;
        o.state = st;
      }
      __syncthreads();
      o2 = uni(s.bin[1]);
      down = b2 < kNT && shift > 0 && o2.cnt >= 2;
      int Eb = E < 0 ? b1 : E;
      if (b1 < 0) {
        if (down || !have || rounded) break;
        Eb = aE;  // the answer of a level above stands
      }
      const BinOut o1 = uni(b1 < 0 ? s.ans : s.bin[0]);
      const bool round = b1 < 0 || o1.state != 1 || !down;
      if (round) {
        const double S1 = exact_sum(s, Eb, o1.part);
        double S2 = 0.0, lhs, right;
        if constexpr (VAR) S2 = exact_sum_sq(s, Eb, o1.ph, o1.pl);
        const bool pass = criterion<VAR>(B, A2, nnz - o1.below, o1.mx, S1, S2, lhs, right);
        if (b1 >= 0 && o1.state == 2 && !pass) {
          // the answer so far and its sums stand
          if (t == b1) st = 0;
          continue;
        }
        T1 = S1;
        rhs = right;
      }
      rounded = round;
      if (t == 0) s.ans = o1;
      have = true;
      aE = Eb;
      break;
    }
    if (!down) break;
    below = o2.below - o2.cnt;
    bsig = o2.part - o2.sig;
    bh = o2.ph - o2.sh;
    bl = o2.pl - o2.sl;
    if (E < 0) {
      E = b2;
      lo = (uint32_t)b2 << 23;
    } else {
      lo += (uint32_t)b2 << shift;
    }
    shift = shift > 9 ? shift - 9 : 0;
    if (!L.lspan)
      request<VAR>(a, s, ctl, sc, row, base, len, L, o2.cnt <= kListCap ? kReqList : kReqWindow, lo, shift, o2.cnt);
  }
  if (!have) {
    // variance budget: no value passes (possible only through rounding with eps = 0), every nonzero
    // is capped
    lam = VAR ? (double)INFINITY : (double)NAN;
    tcap = VAR ? 1u : kKeyInf;
    return VAR ? 0u : (uint32_t)kFlagInternal;
  }
  __syncthreads();
  const BinOut o = uni(s.ans);
  lam = VAR ? T1 / rhs : (B - (double)(nnz - o.below)) / T1;
  tcap = capped_threshold(lam, o.mx + 1);
  return 0;
}

// Algorithm 3 in scale form: lambda_{j+1} = (B - k_j) / U_j, stop when it does not grow. The count
// k_j and the sum U_j of the rest follow from the binades unless the threshold cuts a binade's keys.
GS_DI void solve_greedy(const Args& a, SolveLds<false>& s, RowCtl* ctl, RowScratch* sc, int64_t row, int64_t base,
                        int64_t len, Lead& L, double B, uint64_t nnz, int T, double& lam, uint32_t& tcap) {
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  uint32_t pc = wave_incl(t < kB1 ? s.cnt[t] : 0u, lane);
  if (lane == 63) s.rc[wv] = pc;
  __syncthreads();
  for (int i = 0; i < wv; ++i) pc += s.rc[i];
  if (t < kB1) s.pc[t] = pc;
  // step -1: lambda_0 = B / S
  int e = 254;
  uint64_t K = 0, part = s.sig[254];
  uint32_t q = kKeyInf;  // a first lambda that underflows to zero caps nothing
  lam = 0.0;
#pragma unroll 1
  for (int it = -1;; ++it) {
    const double U = exact_sum(s, e, part);
    if (U == 0.0) break;
    const double ln = (B - (double)K) / U;
    if (!(ln > lam)) break;
    lam = ln;
    q = cap_key(lam);
    if (it + 1 >= T) break;
    e = (int)(q >> 23);
    const uint32_t cnt = s.cnt[e];
    K = nnz - s.pc[e];  // keys >= q, and binade e's significands below q
    part = s.sig[e];
    if ((q & 0x7FFFFFu) == 0) {
      K += cnt;
      part = 0;
    } else if (cnt != 0 && s.mx[e] >= q) {
      uint64_t qc, qs;
      count_above(a, s, ctl, sc, row, base, len, L, q, qc, qs);
      K += qc;
      part -= qs;
    }
  }
  tcap = q;
}

// The leader of a row.
template <int SOLVER, bool VAR = SOLVER == GSPAR_VARIANCE>
GS_DI void lead_row(const Args& a, SolveLds<VAR>& s, RowCtl* ctl, RowScratch* sc, int64_t row, int64_t base,
                    int64_t len) {
  const int t = threadIdx.x;
  const double B = ctl->B;
  const int T = ctl->T;
  uint32_t flags = ctl->flags;
  Lead L;
  // level 1: the copies of the row's histogram summed, one binade per thread
  const Hist1* h = h1_of(a, row);
  uint64_t cnt = 0;
  if (t < kB1) {
    uint64_t sig = 0;
    uint32_t mx = 0;
#pragma unroll
    for (int k = 0; k < kC1; ++k) {
      cnt += h[k].cnt[t];
      sig += h[k].sig[t];
      mx = max(mx, h[k].mx[t]);
    }
    s.cnt[t] = (uint32_t)cnt;
    s.sig[t] = sig;
    s.mx[t] = mx;
    if constexpr (VAR) {
      const H1Q* q = h1q_of(a, row);
      uint64_t qh = 0, ql = 0;
#pragma unroll
      for (int k = 0; k < kC1; ++k) {
        qh += q[k].qh[t];
        ql += q[k].ql[t];
      }
      s.qh[t] = qh;
      s.ql[t] = ql;
    }
  }
  // the candidate band is usable only if every key in it was kept (a statistics workgroup whose
  // region overflowed reserves more than the list holds)
  if (a.lay.cand_cap) {
    L.cand_n = ccnt_of(a, row)->v;
    L.blo = ctl->band_lo;
    L.bhi = ctl->band_hi;
    L.banded = L.cand_n <= (uint64_t)a.lay.cand_cap;
    if (!L.banded) L.blo = L.bhi = 0;
  }
  // the nonzero keys of the row (binade 255 holds only Inf and NaN)
  uint32_t nz = (uint32_t)cnt;
  for (int o = 32; o > 0; o >>= 1) nz += __shfl_xor(nz, o);
  if ((t & 63) == 0) s.rc[t >> 6] = nz;
  if (t == 0) s.err = 0;
  __syncthreads();
  uint64_t nnz = 0;
#pragma unroll
  for (int i = 0; i < kNT / 64; ++i) nnz += s.rc[i];
  nnz = uni(nnz);
  const uint32_t odd = uni(s.cnt[255]);
  __syncthreads();
  double lam = NAN;
  uint32_t tcap = kKeyInf;
  if (odd) flags |= GSPAR_FLAG_NONFINITE;
  if (flags & (GSPAR_FLAG_NONFINITE | GSPAR_FLAG_BADRHO | GSPAR_FLAG_BADSEG)) {
    // no solution: reported, not sampled
  } else if (nnz == 0) {
    flags |= GSPAR_FLAG_ALLZERO;
    lam = INFINITY;
    tcap = 1;
  } else if (!VAR && B >= (double)nnz) {
    lam = INFINITY;
    tcap = 1;
  } else if (!VAR && B == 0.0) {
    lam = 0.0;
  } else {
    if constexpr (SOLVER == GSPAR_GREEDY) {
      solve_greedy(a, s, ctl, sc, row, base, len, L, B, nnz, T, lam, tcap);
    } else {
      double A2 = 0.0;
      if constexpr (VAR) A2 = exact_sum_sq(s, 254, s.qh[254], s.ql[254]);
      flags |= solve_levels<VAR>(a, s, ctl, sc, row, base, len, L, B, nnz, A2, lam, tcap);
    }
    flags |= s.err;  // (the sums end with a barrier)
  }
  if (t == 0) {
    st_agent(&ctl->req, (uint64_t)kReqDone << 32);
    ctl->lam = lam;
    ctl->tcap = tcap;
    ctl->inv_lam = (lam > 0.0 && lam < INFINITY) ? (float)(1.0 / lam) : 0.0f;
    ctl->flags = flags;
    ctl->done = 1;
    ctl->src = L.from;
    ctl->band_lo = L.blo;
    ctl->band_hi = L.bhi;
    ctl->cand_n = L.cand_n;
  }
}

// ------------------------------------------------------------------------------------------
// Kernels.
// ------------------------------------------------------------------------------------------
// Workgroups that fill a segmented call's maps: the 2,150 entries of a residual network's 54 layers took
// one workgroup most of k_init's 10.4 us; with 16 of them k_init takes 6.3.
constexpr int kMapGroups = 16;
// Segmented calls: the workgroup maps of the histogram passes (row << 32 | block) and of the sample
// pass (row << 32 | workgroup within the row), built by up to kMapGroups workgroups of 256 threads
// from the device offsets in row order, 256 rows at a time: an exclusive scan of the per-row counts
// (every workgroup makes it), then every thread fills map entries, finding each entry's row by a binary
// search of the scan. Also the verdict whether the maps have exactly the launched (host) shape.
__device__ void seg_maps(const Args& a, int part, int parts) {
  __shared__ int64_t s_tot[2][4];
  __shared__ int64_t s_pre[2][257];  // exclusive prefixes of the batch's rows (+ the batch total)
  uint64_t* bmap = reinterpret_cast<uint64_t*>(a.ws + a.lay.bmap);
  uint64_t* tmap = reinterpret_cast<uint64_t*>(a.ws + a.lay.tmap);
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  int64_t cb = 0, cw = 0;  // workgroups of the rows before this batch
  for (int64_t r0 = 0; r0 < a.rows; r0 += 256) {
    const int64_t r = r0 + t;
    int64_t nb = 0, nw = 0;
    if (r < a.rows) {
      int64_t base, len;
      row_span(a, r, base, len);
      // 32-bit divisions: a row is shorter than 2^31, a chunk than 2^20
      nb = ((uint32_t)len + (uint32_t)a.chunk - 1u) / (uint32_t)a.chunk;
      const uint32_t rt = len > kTileElems ? (uint32_t)((len + kTileElems - 1) / kTileElems) : 1u;
      nw = (rt + (uint32_t)a.seg_k - 1u) / (uint32_t)a.seg_k;
    }
    int64_t xb = nb, xw = nw;  // inclusive scans over the wave
    for (int o = 1; o < 64; o <<= 1) {
      const int64_t yb = __shfl_up(xb, o), yw = __shfl_up(xw, o);
      if (lane >= o) {
        xb += yb;
        xw += yw;
      }
    }
    if (lane == 63) {
      s_tot[0][wv] = xb;
      s_tot[1][wv] = xw;
    }
    __syncthreads();
    int64_t pb = xb - nb, pw = xw - nw, tb = 0, tw = 0;
    for (int w = 0; w < 4; ++w) {
      if (w < wv) {
        pb += s_tot[0][w];
        pw += s_tot[1][w];
      }
      tb += s_tot[0][w];
      tw += s_tot[1][w];
    }
    s_pre[0][t] = pb;
    s_pre[1][t] = pw;
    if (t == 0) {
      s_pre[0][256] = tb;
      s_pre[1][256] = tw;
    }
    __syncthreads();
    // entry e of the batch belongs to the last row whose prefix is <= e (rows past the end have
    // no entries and the prefix of a row with none equals the next row's)
    for (int m = 0; m < 2; ++m) {
      const int64_t tot = s_pre[m][256], c0 = m == 0 ? cb : cw, cap = m == 0 ? a.seg_blocks : a.seg_wgs;
      uint64_t* map = m == 0 ? bmap : tmap;
      for (int64_t e = t + 256 * part; e < tot && c0 + e < cap; e += 256 * parts) {
        int lo = 0, hi = 255;  // the row lies in [lo, hi]
        while (lo < hi) {
          const int mid = (lo + hi + 1) >> 1;
          if (s_pre[m][mid] <= e) lo = mid;
          else hi = mid - 1;
        }
        map[c0 + e] = ((uint64_t)(r0 + lo) << 32) | (uint64_t)(e - s_pre[m][lo]);
      }
    }
    cb += tb;
    cw += tw;
    __syncthreads();
  }
  if (part == 0 && t == 0) *segok_of(a) = (cb == a.seg_blocks && cw == a.seg_wgs) ? 1u : 2u;
}

__global__ void __launch_bounds__(256) k_init(Args a) {
  if (a.seg && blockIdx.x < kMapGroups) seg_maps(a, (int)blockIdx.x, (int)min(gridDim.x, (uint32_t)kMapGroups));
  const int64_t tid = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  // level-1 histogram copies, capped-count lines, look-back status words
  uint64_t* h1 = reinterpret_cast<uint64_t*>(a.ws + a.lay.h1);
  const int64_t n1 = a.rows * kC1 * (int64_t)(sizeof(Hist1) / 8);
  for (int64_t i = tid; i < n1; i += stride) h1[i] = 0;
  uint64_t* kc = reinterpret_cast<uint64_t*>(a.ws + a.lay.kc);
  const int64_t nkc = (int64_t)((a.lay.status - a.lay.kc) / 8);
  for (int64_t i = tid; i < nkc; i += stride) kc[i] = 0;
  uint64_t* st = status_of(a);
  const int64_t ns = a.rows * a.lay.tiles;
  for (int64_t i = tid; i < ns; i += stride) st[i] = 0;
  if (a.solver == GSPAR_VARIANCE) {
    uint64_t* q = reinterpret_cast<uint64_t*>(a.ws + a.lay.h1q);
    const int64_t nq = a.rows * kC1 * (int64_t)(sizeof(H1Q) / 8);
    for (int64_t i = tid; i < nq; i += stride) q[i] = 0;
  }
  if (a.lay.cand_cap) {
    // sample histograms and candidate count lines (adjacent in the layout)
    uint64_t* pc = reinterpret_cast<uint64_t*>(a.ws + a.lay.pre);
    const int64_t np = (int64_t)((a.lay.cand - a.lay.pre) / 8);
    for (int64_t i = tid; i < np; i += stride) pc[i] = 0;
  }
  for (int64_t r = tid; r < a.rows; r += stride) {
    RowCtl c;
    memset(&c, 0, sizeof(c));
    const double rho = a.rho_dev ? a.rho_dev[r] : a.rho;
    int64_t base, len;
    const bool ok = row_span(a, r, base, len);
    if (a.solver == GSPAR_VARIANCE) {
      // the variance budget eps (any finite eps >= 0) in place of the density
      c.B = rho;
      if (!(rho >= 0.0 && rho < INFINITY)) c.flags = GSPAR_FLAG_BADRHO;
    } else {
      c.B = rho * (double)len;
      if (!(rho >= 0.0 && rho <= 1.0)) c.flags = GSPAR_FLAG_BADRHO;
    }
    if (!ok) c.flags |= GSPAR_FLAG_BADSEG;
    c.solver = a.solver;
    c.T = a.T;
    *ctl_of(a, r) = c;
  }
}

// Row and block of a histogram-pass workgroup: rows * nb workgroups for a strided batch, the map
// built by k_init for a segmented call (false: nothing to do).
__device__ __forceinline__ bool hist_block(const Args& a, int64_t& row, int64_t& blk) {
  if (!a.seg) {
    row = blockIdx.x / a.nb;
    blk = blockIdx.x % a.nb;
    return true;
  }
  if (*segok_of(a) != 1) return false;
  const uint64_t e = reinterpret_cast<const uint64_t*>(a.ws + a.lay.bmap)[blockIdx.x];
  row = (int64_t)(e >> 32);
  blk = (int64_t)(e & 0xFFFFFFFFu);
  return true;
}

// A global-memory pointer every lane holds equally, moved to scalar registers (on the device:
// in the global address space, so stores take a scalar base and a 32-bit vector offset).
#if defined(__HIP_DEVICE_COMPILE__)
typedef __attribute__((address_space(1))) char gchar;
#define GS_GLOBAL(T) T __attribute__((address_space(1)))
__device__ __forceinline__ gchar* uniform_ptr(void* p) {
  const uint64_t u = (uint64_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)u);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(u >> 32));
  return (gchar*)(((uint64_t)hi << 32) | lo);
}
#else
typedef char gchar;
#define GS_GLOBAL(T) T
GS_HD gchar* uniform_ptr(void* p) { return static_cast<gchar*>(p); }
#endif

// Systematic sample of each row for the candidate band: kPreWG workgroups per row each read
// kPreLines of the row's whole 64-byte lines, spread evenly over the row, and add a histogram over
// binades (count, significand sum) into the row's PreHist. Every load is issued before any is used.
__global__ void __launch_bounds__(256) k_presample(Args a) {
  static_assert(kB1 == 256 && kPreLines % 64 == 0, "one binade per thread, 64 lines per round");
  constexpr int kRounds = kPreLines / 64;
  constexpr int kCopies = 4;  // LDS copies by lane, to spread same-bin atomics
  __shared__ uint32_t s_cnt[kB1 * kCopies];
  __shared__ unsigned long long s_sig[kB1 * kCopies];
  const int64_t row = blockIdx.x / kPreWG;
  const int p = (int)(blockIdx.x % kPreWG);
  const int t = threadIdx.x;
  for (int i = t; i < kB1 * kCopies; i += 256) {
    s_cnt[i] = 0;
    s_sig[i] = 0;
  }
  __syncthreads();
  const float* __restrict__ gr = a.g + row * a.ld;
  const int64_t nl = a.d / 16;         // whole lines of the row
  const int64_t ns = pre_lines(a.d);   // lines sampled (ns <= nl)
  float4 x[kRounds];
#pragma unroll
  for (int j = 0; j < kRounds; ++j) {
    const int64_t i = (int64_t)p * kPreLines + j * 64 + (t >> 2);  // sample index
    const int64_t line = (i < ns ? i : ns - 1) * nl / ns;             // < nl
    x[j] = load_vec(gr + 16 * line + 4 * (t & 3));
  }
  __builtin_amdgcn_sched_barrier(0);
  const int lc = t & (kCopies - 1);
#pragma unroll
  for (int j = 0; j < kRounds; ++j) {
    const int64_t i = (int64_t)p * kPreLines + j * 64 + (t >> 2);
    if (i >= ns) continue;  // past the sample (rows with fewer lines than a full sample)
    const float v[4] = {x[j].x, x[j].y, x[j].z, x[j].w};
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const uint32_t key = key_of(v[c]);
      if (key != 0) {
        const uint32_t b = (key >> 23) * kCopies + lc;
        atomicAdd(&s_cnt[b], 1u);
        atomicAdd(&s_sig[b], (unsigned long long)key_sig(key));
      }
    }
  }
  __syncthreads();
  uint64_t cnt = 0, sg = 0;
#pragma unroll
  for (int k = 0; k < kCopies; ++k) {
    cnt += s_cnt[t * kCopies + k];
    sg += s_sig[t * kCopies + k];
  }
  if (cnt) {
    PreHist* h = pre_of(a, row);
    atomicAdd((unsigned long long*)&h->cnt[t], (unsigned long long)cnt);
    atomicAdd((unsigned long long*)&h->sig[t], (unsigned long long)sg);
  }
}

// LDS of the band prediction.
struct BandLds {
  double w[kNT / 64];
  uint64_t k[kNT / 64];
  int ired[kNT / 64];
  double ge;   // the sample's G at the lower edge of the binade of 1/lambda*
  double ge1;  // and at the lower edge of the next binade up
};
// G within this fraction of B at that edge: 1/lambda* may lie in the binade below.
constexpr double kBandNear = 0.125;

// The candidate band of a row, predicted from its sample histogram identically by every
// workgroup of the statistics pass (same data, same order of operations). With f = the row's
// length over the sampled count, the sums are scaled sample sums. Every threshold a solver will
// refine lies in [1/lambda*, 1/lambda_0]: 1/lambda_0 = S / B (Algorithm 3's start), and the exact
// 1/lambda* is where G(tau) = #{a >= tau} + (sum of the a < tau) / tau falls to B (Proposition 1:
// sum min(lambda a, 1) = B); G decreases in tau, so at binade edges its crossing gives the binade
// e* of 1/lambda*. The exact solver refines the binade of 1/lambda*, or the next occupied one
// above it when no key of that binade lies above 1/lambda* (only when the crossing is at its top),
// so its band is e*, with e* - 1 or e* + 1 too when the sample's G at e*'s lower or upper edge is
// within kBandNear of B (the sample may have misplaced the crossing); the greedy solver's
// thresholds run from 1/lambda_0 = S / B down towards 1/lambda*, so its band reaches up to the
// binade of 1.25 S / B (slack for the sample's estimate of S). Whole binades, so every refinement
// window inside the band is complete. No band when B = 0 or nothing was sampled. Threads 0..255
// own one binade each; every thread receives the result.
GS_DI void cand_band(const Args& a, const PreHist* ph, double B, int64_t len, BandLds& sm, uint32_t& blo,
                     uint32_t& bhi) {
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  uint64_t c = 0;
  double w = 0.0;
  if (t < kB1) {
    c = ph->cnt[t];
    w = c ? ldexp((double)ph->sig[t], binade_shift(t) - 149) : 0.0;
  }
  // inclusive suffix sums over binades (count and value sum of the binades >= t)
  uint64_t kc = c;
  double wc = w;
  for (int o = 1; o < 64; o <<= 1) {
    const uint64_t ky = __shfl_down(kc, (unsigned)o);
    const double wy = __shfl_down(wc, (unsigned)o);
    if (lane + o < 64) {
      kc += ky;
      wc += wy;
    }
  }
  if (lane == 0) {
    sm.k[wv] = kc;
    sm.w[wv] = wc;
  }
  __syncthreads();
  double tot = 0.0;
  for (int i = 0; i < kB1 / 64; ++i) tot += sm.w[i];
  for (int i = wv + 1; i < kB1 / 64; ++i) {
    kc += sm.k[i];
    wc += sm.w[i];
  }
  const double f = (double)len / (16.0 * (double)pre_lines(len));
  // the highest occupied binade of the sample
  int top = (t < kB1 - 1 && c) ? t : -1;
  for (int o = 32; o > 0; o >>= 1) top = max(top, __shfl_xor(top, o));
  if (lane == 0) sm.ired[wv] = top;
  __syncthreads();
  top = -1;
  for (int i = 0; i < kNT / 64; ++i) top = max(top, sm.ired[i]);
  __syncthreads();
  int best = -1;
  double G = 0.0;
  if (t >= 1 && t < kB1 - 1 && B > 0.0 && tot > 0.0) {
    // G at the binade's lower edge lo = 2^(t - 127): keys >= lo count whole, the rest by value / lo
    const double lo = ldexp(1.0, t - 127);
    G = f * ((double)kc + (tot - wc) / lo);
    if (G >= B) best = t;
  }
  for (int o = 32; o > 0; o >>= 1) best = max(best, __shfl_xor(best, o));
  if (lane == 0) sm.ired[wv] = best;
  __syncthreads();
  int e = -1;
  for (int i = 0; i < kNT / 64; ++i) e = max(e, sm.ired[i]);
  if (t == e) sm.ge = G;
  if (t == e + 1) sm.ge1 = G;
  __syncthreads();
  blo = bhi = 0;
  // Nothing looks capped (B times the sample's largest magnitude, bounded by its binade's top,
  // below half the estimated sum): the solvers should need no window, so no band is collected (a
  // row the sample misjudged refines over the row).
  const bool uncapped = top >= 0 && B * ldexp(1.0, top - 126) <= 0.5 * f * tot;
  if (e >= 1 && B > 0.0 && tot > 0.0 && !uncapped) {
    const uint32_t elo = (uint32_t)e - (sm.ge < (1.0 + kBandNear) * B ? 1u : 0u);
    uint32_t ehi = (uint32_t)e + (sm.ge1 >= (1.0 - kBandNear) * B ? 1u : 0u);
    if (a.solver == GSPAR_GREEDY) {
      const double t0 = 1.25 * f * tot / B;
      const uint32_t e0 = t0 < 3.0e38 ? (key_of((float)t0) >> 23) : 254u;
      ehi = e0 > ehi ? e0 : ehi;
    }
    blo = elo << 23;
    bhi = (ehi + 1) << 23;
    if (bhi > kKeyInf) bhi = kKeyInf;
  }
  __syncthreads();
}

// Streaming statistics pass. Grid: rows * nb workgroups of kNT threads. Each builds an LDS
// histogram over binades (count, exact significand sum, maximum key), kept in kLaneCopies copies
// by lane to spread same-address LDS atomics, and adds its nonempty bins into one of the row's kC1
// global copies (chosen by workgroup index) with atomics. k_solve runs next.
template <bool SQ, bool CAND>
__global__ void __launch_bounds__(kNT) __attribute__((amdgpu_waves_per_eu(4))) k_stats(Args a) {
  __shared__ StatsLdsT<SQ> sm_st;
  StatsLdsT<SQ>& sm = sm_st;
  __shared__ BandLds s_band;
  // candidate band: per-wave buffers of collected keys, and the workgroup's region count
  __shared__ uint32_t s_cand[CAND ? kNT / 64 : 1][CAND ? 64 * kCandLane : 1];
  __shared__ uint32_t s_rcnt;
  __shared__ unsigned long long s_rbase;
  int64_t row, blk;
  if (!hist_block(a, row, blk)) return;
  int64_t base, len;
  row_span(a, row, base, len);
  const int64_t beg = blk * a.chunk;
  if (beg >= len) return;  // past the end of a shorter segment
  uint32_t blo = 0, bhi = 0;
  if constexpr (CAND) {
    cand_band(a, pre_of(a, row), ctl_of(a, row)->B, len, s_band, blo, bhi);
    if (blk == 0 && threadIdx.x == 0) {
      RowCtl* c = ctl_of(a, row);
      c->band_lo = blo;
      c->band_hi = bhi;
    }
  }
  // zero keys are never candidates (no window counts them): the band starts at key 1 at least
  const uint32_t blo1 = blo ? blo : 1u;
  const uint32_t bspan = bhi > blo1 ? bhi - blo1 : 0u;
  const int lane = threadIdx.x & 63;
  // Collected keys are buffered per lane in LDS (kCandLane slots, no cross-lane work per group).
  // When some lane could not take a whole group's keys the wave flushes every lane's buffer into
  // this workgroup's own region of the row's candidate buffer, at a place taken from an LDS
  // counter, lanes in order by a wave prefix; keys that would pass the region's end are dropped and
  // the region is marked overflowed, so the solver does not use the band.
  uint32_t* const lbuf = &s_cand[CAND ? threadIdx.x >> 6 : 0][CAND ? lane * kCandLane : 0];
  uint32_t lcnt = 0;
  if (CAND && threadIdx.x == 0) s_rcnt = 0;
  auto flush = [&]() {
    uint32_t wtot;
    const uint32_t pre = wave_prefix_bits<3>(lcnt, wtot);
    uint32_t b0 = 0;
    if (lane == 0) b0 = atomicAdd(&s_rcnt, wtot);
    const uint32_t b = (uint32_t)__shfl((int)b0, 0) + pre;
    uint32_t* __restrict__ dst = creg_of(a, row) + blk * a.cand_region;
    for (uint32_t j = 0; j < lcnt; ++j)
      if ((int64_t)b + j < a.cand_region) dst[b + j] = lbuf[j];
    lcnt = 0;
  };
  for (int b = threadIdx.x; b < kB1 * kLaneCopies; b += kNT) {
    sm.pk[b] = 0;
    sm.mx[b] = 0;
    if constexpr (SQ) {
      sm.qh[b] = 0;
      sm.ql[b] = 0;
    }
  }
  __syncthreads();
  const float* __restrict__ gr = a.g + base;
  const int64_t end = min(len, beg + a.chunk);
  const uint32_t lc = threadIdx.x & (kLaneCopies - 1);
  auto hist = [&](const float v[4]) {
    // the group's additions first (atomics without return), then its four bin maxima read
    // together: one LDS round trip per group. The bin maximum only grows, so a read that already
    // covers the key skips the atomic. Zero keys (also the coordinates outside [beg, end), read as
    // 0) add nothing, and their bin-0 reads are not acted on.
    uint32_t key[4], f[4], cur[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      key[c] = key_of(v[c]);
      f[c] = (key[c] >> 23) * kLaneCopies + lc;
      if (key[c] != 0) {
        atomicAdd(&sm.pk[f[c]], (unsigned long long)((1ull << 44) + key_sig(key[c])));
        if constexpr (SQ) {
          const uint64_t m = key_sig(key[c]), m2 = m * m;
          atomicAdd(&sm.qh[f[c]], (unsigned long long)(m2 >> 24));
          atomicAdd(&sm.ql[f[c]], (unsigned long long)(m2 & 0xFFFFFFu));
        }
      }
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) cur[c] = sm.mx[f[c]];
#pragma unroll
    for (int c = 0; c < 4; ++c)
      if (key[c] > cur[c]) atomicMax(&sm.mx[f[c]], key[c]);
  };
  // the candidate band's keys of a group into the lane's buffer (room for four made first); a wave
  // whose groups all lie below the band (most of them) skips the group
  auto collect = [&](const float v[4]) {
    const uint32_t kmax = max(max(key_of(v[0]), key_of(v[1])), max(key_of(v[2]), key_of(v[3])));
    if (!__ballot(kmax >= blo1)) return;
    if (__ballot(lcnt > (uint32_t)(kCandLane - 4))) flush();
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const uint32_t key = key_of(v[c]);
      if (key - blo1 < bspan) lbuf[lcnt++] = key;
    }
  };
  // rows long enough for a candidate band (2^25 coordinates and more) keep 8 loads per lane in flight,
  // shorter ones 4 (on 2^28 coordinates 8 save about 4 microseconds per pass; on 2.5 * 10^7 and
  // fewer they cost 1-3)
  constexpr int kU = CAND ? 8 : 4;
  if (CAND && bspan != 0) {
    stream_groups<kU, kNT>(gr, beg, end, [&](int64_t, const float v[4], uint32_t) {
      hist(v);
      collect(v);
    });
  } else {
    // no band (or none predicted for this row): the plain statistics loop
    stream_groups<kU, kNT>(gr, beg, end, [&](int64_t, const float v[4], uint32_t) { hist(v); });
  }
  if constexpr (CAND) {
    if (__ballot(lcnt != 0)) flush();
    __syncthreads();
    // move the region to the row's compact list: one reservation per workgroup (a region that
    // overflowed reserves past the list's capacity, which disables the band)
    if (bspan != 0) {
      const uint32_t n = s_rcnt;
      if (threadIdx.x == 0) {
        const unsigned long long want = (int64_t)n <= a.cand_region ? n : (unsigned long long)a.lay.cand_cap + 1;
        s_rbase = want ? atomicAdd(&ccnt_of(a, row)->v, want) : 0ull;
      }
      __syncthreads();
      const uint64_t b = s_rbase;
      if ((int64_t)n <= a.cand_region && b + n <= (uint64_t)a.lay.cand_cap) {
        const uint32_t* __restrict__ src = creg_of(a, row) + blk * a.cand_region;
        uint32_t* __restrict__ out = cand_of(a, row) + b;
        for (uint32_t j = threadIdx.x; j < n; j += kNT) out[j] = src[j];
      }
    }
  }
  __syncthreads();
  // flush one binade per thread into copy (blk mod kC1)
  if (threadIdx.x < kB1) {
    const int e = threadIdx.x;
    uint64_t cnt = 0, sg = 0;
    uint32_t mx = 0;
#pragma unroll
    for (int j = 0; j < kLaneCopies; ++j) {
      const uint64_t p = sm.pk[e * kLaneCopies + j];
      cnt += p >> 44;
      sg += p & ((1ull << 44) - 1);
      mx = max(mx, sm.mx[e * kLaneCopies + j]);
    }
    if (cnt) {
      Hist1* h = h1_of(a, row, (int)(blk % kC1));
      atomicAdd((unsigned long long*)&h->cnt[e], (unsigned long long)cnt);
      atomicAdd((unsigned long long*)&h->sig[e], (unsigned long long)sg);
      atomicMax(&h->mx[e], mx);
      if constexpr (SQ) {
        uint64_t qh = 0, ql = 0;
#pragma unroll
        for (int j = 0; j < kLaneCopies; ++j) {
          qh += sm.qh[e * kLaneCopies + j];
          ql += sm.ql[e * kLaneCopies + j];
        }
        H1Q* q = h1q_of(a, row, (int)(blk % kC1));
        atomicAdd((unsigned long long*)&q->qh[e], (unsigned long long)qh);
        atomicAdd((unsigned long long*)&q->ql[e], (unsigned long long)ql);
      }
    }
  }
}

// The solver. Grid: a leading workgroup per row, then the helpers: a.helpers per row of a strided
// batch; for a segmented call a workgroup per map entry, of which those of every help_step-th block help.
// Two workgroups of it fit a compute unit (128 registers), so that all 512 of 16 rows' are resident:
// with one, under the variance budget, half of the rows had no helpers until the others were solved
// (the kernel took 140 us on 16 rows of 2^20, and takes 65).
template <int SOLVER>
__global__ void __launch_bounds__(kNT, 4) k_solve(Args a) {
  constexpr bool VAR = SOLVER == GSPAR_VARIANCE;
  __shared__ SolveLds<VAR> sm;
  const bool lead = blockIdx.x < a.rows;
  const int64_t h = (int64_t)blockIdx.x - a.rows;
  int64_t row = blockIdx.x;
  uint32_t help = 0;
  if (a.seg && *segok_of(a) != 1) {
    // the workgroup maps of a segmented call do not have the launched shape: no histogram pass
    // ran and the sample pass does nothing, so the row is skipped and its results written here
    if (lead && threadIdx.x == 0) {
      RowCtl* c = ctl_of(a, row);
      c->flags |= GSPAR_FLAG_BADSEG;
      c->lam = NAN;
      c->tcap = kKeyInf;
      c->inv_lam = 0.0f;
      c->done = 1;
      if (a.nnz) a.nnz[row] = 0;
      if (a.nnz_b) a.nnz_b[row] = 0;
      if (a.inv_out) a.inv_out[row] = 0.0f;
      if (a.k_out) a.k_out[row] = 0;
      if (a.lam_out) a.lam_out[row] = NAN;
      if (a.flags_out) a.flags_out[row] = c->flags;
    }
    return;
  }
  if (!lead) {
    if (!a.seg) {
      row = (uint32_t)h / (uint32_t)a.helpers;
      help = (uint32_t)h % (uint32_t)a.helpers + 1u;
    } else {
      const uint64_t e = reinterpret_cast<const uint64_t*>(a.ws + a.lay.bmap)[h];
      const uint32_t blk = (uint32_t)e;
      if (blk == 0 || blk % (uint32_t)a.help_step != 0) return;
      help = blk / (uint32_t)a.help_step;
      row = (int64_t)(e >> 32);
    }
  }
  int64_t base, len;
  row_span(a, row, base, len);
  if (lead) {
    lead_row<SOLVER>(a, sm, ctl_of(a, row), scratch_of(a, row), row, base, len);
  } else {
    uint32_t helpers = (uint32_t)a.helpers;
    if (a.seg) {  // (32-bit divisions: a row is shorter than 2^31, a chunk than 2^20)
      const uint32_t n = ((uint32_t)len + (uint32_t)a.chunk - 1u) / (uint32_t)a.chunk;
      helpers = (n - 1u) / (uint32_t)a.help_step;
    }
    help_row<VAR>(a, sm, ctl_of(a, row), scratch_of(a, row), row, base, len, help, helpers);
  }
}

// Sampling, amplification and order-preserving compaction. Workgroup t handles tile t (kTileElems
// coordinates of one row, in row order); wave w of the workgroup owns the tile's w-th quarter and
// reads it as kTileGroups coalesced float4 loads per lane. Tile prefixes chain through a decoupled
// look-back whose status word packs (flag:2 | capped survivors:31 | survivors:31). A predecessor
// that has not published after a long back-off is counted by the waiting wave itself, so no
// ordering of workgroup dispatch is assumed and every wait ends.
constexpr uint64_t kStAgg = 1ull << 62, kStInc = 2ull << 62, kStVal = (1ull << 62) - 1;
// Look-back rounds before a waiting wave counts an unpublished predecessor itself (a build may
// lower it to exercise that path).
#ifndef GSPAR_LOOKBACK_POLLS
#define GSPAR_LOOKBACK_POLLS 4096
#endif
constexpr int kPolls = GSPAR_LOOKBACK_POLLS;
constexpr int kWaveElems = kTileElems / (kTileThreads / 64);  // coordinates per wave per tile

struct TileCtx {
  const float* row;
  int64_t d;
  double lam;
  uint32_t tcap;
  uint32_t k0, k1;
  bool live;
};

// Selection bits (bit c: coordinate 4q+c survives) and capped-survivor bits of group q, whose
// values v are given (m: bit c set when coordinate 4q+c exists).
__device__ __forceinline__ void decide_values(const TileCtx& c, int64_t q, const float v[4], uint32_t m, uint32_t& z,
                                              uint32_t& cz) {
  uint32_t x0 = (uint32_t)q, x1 = (uint32_t)((uint64_t)q >> 32), x2 = 0, x3 = 0;
  philox10(x0, x1, x2, x3, c.k0, c.k1);
  const uint32_t xr[4] = {x0, x1, x2, x3};
  z = 0;
  cz = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint32_t key = key_of(v[k]);
    const bool capped = key >= c.tcap;
    const bool pick = capped || ((double)xr[k] * 0x1p-32 < c.lam * (double)fabsf(v[k]));
    const bool sel = c.live && ((m >> k) & 1) && key != 0 && pick;
    z |= (uint32_t)sel << k;
    cz |= (uint32_t)(sel && capped) << k;
  }
}

// The same for group q loaded here (entries past the row's end read as 0).
__device__ __forceinline__ void decide_group(const TileCtx& c, int64_t q, float v[4], uint32_t& z, uint32_t& cz) {
  const uint32_t m = load4(c.row, q, c.d, v);
  decide_values(c, q, v, m, z, cz);
}

// Aggregate (capped << 31 | survivors) of tile `part` computed by one wave (fallback path).
__device__ uint64_t wave_tile_aggregate(const TileCtx& c, int64_t part, int lane) {
  uint64_t n = 0, nc = 0;
  for (int j = 0; j < kTileElems / 4 / 64; ++j) {
    const int64_t q = part * (kTileElems / 4) + j * 64 + lane;
    float v[4];
    uint32_t z, cz;
    decide_group(c, q, v, z, cz);
    n += __popc(z);
    nc += __popc(cz);
  }
  for (int o = 32; o > 0; o >>= 1) {
    n += __shfl_xor(n, o);
    nc += __shfl_xor(nc, o);
  }
  return (nc << 31) | n;
}

// Phase 1: each lane decides kTileGroups groups of its wave's quarter (coalesced loads, one
// Philox block per group) and writes one byte per group to LDS: selection bits (low nibble) and
// sign bits (high nibble); capped survivors (emitted unscaled) append their value to the deciding
// lane's own LDS row, and a second byte array holds per group their bits and the lane's running
// count of them. The wave totals give the tile aggregate, published at once; wave 0 then looks back
// for the tile's prefix.
// Phase 2: thread t owns the tile's groups [16t, 16t + 16), i.e. 64 consecutive coordinates
// inside its own wave's quarter, so its survivors are contiguous in the output: one prefix over
// the wave's lanes places it, and it writes only its own set bits, through an LDS staging area of
// kStageEmit survivors that the wave then stores with consecutive lanes on consecutive slots (up to
// kDenseEmit survivors of its 4,096; rows of the variance budget that keep a quarter of 16 x 2^20
// coordinates take 37 us this way against 63 with one store per lane and survivor). Phase 2 reads no
// global memory (a load would wait for every store issued before it), except in a wave where some lane
// kept more capped values than its LDS row holds (a separate instantiation).
// Capped survivors' values are kept in LDS by the phase-1 lane that decided them, kLaneCap per
// lane and tile (rows padded to kLaneStride floats so that lanes fall on different banks); a wave
// with a lane past that reads its capped values from global memory in phase 2.
// A group with one capped coordinate (nearly all that have any) keeps its largest magnitude, known
// already, in one store: on 2^28 coordinates with one per cent of outliers, at rho = 0.1, the pass takes
// 274 us against 280 with a store for each of the four.
constexpr int kLaneCap = 8;
constexpr int kLaneStride = kLaneCap + 1;
constexpr int kSampleBatch = 8;  // float4 loads in flight per lane in the sampling pass
// Survivors of a wave's quarter tile (of 4096) above which emission goes by groups: the staged loops take
// as many steps as the fullest lane of each round, which grows with the square of the density.
constexpr int kDenseEmit = 2048;
// The compaction of a wave that has more capped survivors on a lane than its LDS row holds goes by groups
// above kGroupEmit survivors of which more than kGroupCapped are capped: its other choice stores one
// survivor per lane and step and reads every capped one from g, and each read waits for the stores
// before it (by groups, one read serves a group). us a call by groups and one by one, with the capped
// survivors of a wave: 16 x 2^20 Student-t(2) rows, greedy, 97 and 95 at 164, 107 and 118 at 213, 119
// and 315 at 352; 2^26 coordinates 247 and 241 at 164, 348 and 393 at 213, 369 and 1,076 at 352; normal
// rows under the variance budget (eps = 0.5) 151 and 407 at 303. Where all survivors are capped: 16 x
// 2^20 72 and 70 at 328, 70 and 77 at 369, 70 and 98 at 492, 2^26 238 and 230, 237 and 250, 238 and 326.
constexpr int kGroupEmit = 352;
constexpr int kGroupCapped = 192;
// Survivors staged in LDS at a time: 4-byte entries in the quarter's 2 KB of code and capped-survivor
// bytes, free once every lane has read its own.
constexpr int kStageEmit = 512;
static_assert(kTileGroups % kSampleBatch == 0 && kTileGroups == 16, "tile shape");
static_assert(2 * kStageEmit <= kWaveElems / 4 && kTileElems <= 65536 && 64 * kLaneStride <= 1024,
              "a staged entry: 16-bit tile coordinate, 10-bit capped-value place, within the quarter's bytes");
// Below this lambda, lambda * 2^32 * |g| could round differently from (lambda * |g|) * 2^32.
constexpr double kLamScaledMin = 0x1p-900;

// The smallest and the largest of four magnitudes (one three-input and one two-input instruction;
// written out because the library functions first quiet every operand).
__device__ __forceinline__ float min_abs4(const float d[4]) {
#if defined(__HIP_DEVICE_COMPILE__)
  float r;
  asm("v_min3_f32 %0, |%1|, |%2|, |%3|" : "=v"(r) : "v"(d[0]), "v"(d[1]), "v"(d[2]));
  asm("v_min_f32 %0, %0, |%1|" : "+v"(r) : "v"(d[3]));
  return r;
#else
  return min(min(fabsf(d[0]), fabsf(d[1])), min(fabsf(d[2]), fabsf(d[3])));
#endif
}
__device__ __forceinline__ float max_abs4(const float d[4]) {
#if defined(__HIP_DEVICE_COMPILE__)
  float r;
  asm("v_max3_f32 %0, |%1|, |%2|, |%3|" : "=v"(r) : "v"(d[0]), "v"(d[1]), "v"(d[2]));
  asm("v_max_f32 %0, %0, |%1|" : "+v"(r) : "v"(d[3]));
  return r;
#else
  return max(max(fabsf(d[0]), fabsf(d[1])), max(fabsf(d[2]), fabsf(d[3])));
#endif
}
// The sign bits of four floats, bit k of byte k of `mask` where float k is negative: v_perm_b32's
// sign-replicating selectors (9: bit 31 of the low word of the pair, 11: of the high word) turn each
// sign into a 0x00 / 0xFF byte.
__device__ __forceinline__ uint32_t sign_bytes(const float v[4], uint32_t mask) {
  const uint32_t s01 = __builtin_amdgcn_perm(__float_as_uint(v[1]), __float_as_uint(v[0]), 0x0C0C0B09u);
  const uint32_t s23 = __builtin_amdgcn_perm(__float_as_uint(v[3]), __float_as_uint(v[2]), 0x0B090C0Cu);
  return (s01 | s23) & mask;
}
constexpr uint32_t kSelBytes = 0x08040201u, kSignBytes = 0x80402010u;

// |x| with bit 31 of `s` as its sign.
__device__ __forceinline__ float signed_as(float x, uint32_t s) {
  const uint32_t u = (__float_as_uint(x) & 0x7FFFFFFFu) | (s & 0x80000000u);
  memcpy(&x, &u, 4);
  return x;
}

// What a row's whole tiles are decided with (see decide_fast).
struct FastCtx {
  double lam32;  // lambda * 2^32
  float lamf;    // the same in fp32
  float tol;     // |difference| up to which fp32 does not decide
};
__device__ __forceinline__ FastCtx fast_ctx(double lam) {
  FastCtx f;
  f.lam32 = lam * 0x1p32;
  const bool in = f.lam32 <= 0x1p100;  // beyond, fp32 could overflow: everything is decided in fp64
  f.lamf = in ? (float)f.lam32 : 0x1p100f;
  f.tol = in ? 1024.0f : INFINITY;
  return f;
}

// Whole-tile decisions with the scaled threshold: coordinate i survives iff
// x_i < t_i = fl(lambda * 2^32 * |g_i|), which equals the comparison x_i < fl(lambda * |g_i|) * 2^32
// (exact scaling by a power of two) for lambda = 0 or lambda >= kLamScaledMin.
//
// The pass is bound by instruction issue, so the comparison is made in fp32 first: the difference
// fl(x - lamf |g|) is within 2^-24 x + 2^-23 t + its own rounding of x - t, 1024 in all where x and t are
// at most 2^32 (and t beyond that only makes it more negative), so outside +-1024 its sign decides;
// within (about one wave in eight thousand groups) the group is decided in fp64. Two instructions per
// coordinate and one sign gather per group take the place of five and seven: by this alone the pass went
// from 262 to 241 us on 2^28 coordinates at rho = 0.01, from 310 to 285 at 0.1, and from 20.1 to 19.1
// on 16 x 2^20 (kernel times within a call; from run to run they differ by some 2 per cent).
//
// Returns bit k of byte k for each survivor.
__device__ __forceinline__ uint32_t decide_fast(int64_t q, const float v[4], const FastCtx& f, uint32_t k0,
                                                uint32_t k1) {
  // rows are shorter than 2^31 coordinates, so the counter's high word floor(i/4) >> 32 is 0; with
  // that known the first rounds fold into fewer vector operations
  uint32_t x0 = (uint32_t)q, x1 = 0, x2 = 0, x3 = 0;
  philox10(x0, x1, x2, x3, k0, k1);
  const uint32_t xr[4] = {x0, x1, x2, x3};
  float d[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) d[k] = fmaf(-fabsf(v[k]), f.lamf, (float)xr[k]);
  uint32_t sel = sign_bytes(d, kSelBytes);
  if (__builtin_expect(min_abs4(d) <= f.tol, 0)) {
    sel = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) sel |= (uint32_t)((double)xr[k] < f.lam32 * (double)fabsf(v[k])) << (9 * k);
  }
  return sel;
}

// The nibbles of the eight bytes of (w0, w1), byte 0 of w0 first: lo holds their low nibbles and hi
// their high nibbles, byte k's at bits [4k, 4k + 4). v_perm_b32 gathers the even and the odd bytes
// (selectors 0-7 pick a byte of the pair, w1 above w0), and one bit-field insert interleaves each.
__device__ __forceinline__ void byte_nibbles(uint32_t w0, uint32_t w1, uint32_t& lo, uint32_t& hi) {
  const uint32_t ev = __builtin_amdgcn_perm(w1, w0, 0x06040200u);  // bytes 6, 4, 2, 0
  const uint32_t od = __builtin_amdgcn_perm(w1, w0, 0x07050301u);  // bytes 7, 5, 3, 1
  lo = (ev & 0x0F0F0F0Fu) | ((od << 4) & 0xF0F0F0F0u);
  hi = ((ev >> 4) & 0x0F0F0F0Fu) | (od & 0xF0F0F0F0u);
}

template <bool HYB, int K>
__global__ void __launch_bounds__(kTileThreads) k_sample(Args a) {
  __shared__ float s_capl[K][kTileThreads / 64][64 * kLaneStride];
  __shared__ alignas(16) uint8_t s_code[K][kTileElems / 4];  // per group: selection | sign << 4
  // per group: capped-survivor bits | the deciding lane's capped count before the group << 4
  __shared__ alignas(16) uint8_t s_capb[K][kTileElems / 4];
  __shared__ uint32_t s_wsel[K][kTileThreads / 64];
  __shared__ uint32_t s_wcap[K][kTileThreads / 64];
  __shared__ uint32_t s_wcl[K][kTileThreads / 64];
  __shared__ uint64_t s_excl;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  // workgroup -> K consecutive tiles [part0, part0 + nk) of one row. A row has
  // max(1, ceil(length / kTileElems)) tiles, all lay.tiles for rows of a strided batch; the
  // workgroups past a shorter segment's tiles have nothing to do (no later tile of the row waits on
  // them, and its last tile writes the row's results).
  int64_t row, part0;
  if (!a.seg) {
    const uint32_t wpr = (uint32_t)((a.lay.tiles + K - 1) / K);  // workgroups per row (a row has at most 2^17 tiles)
    row = blockIdx.x / wpr;
    part0 = (int64_t)(blockIdx.x % wpr) * K;
  } else {
    // the map built by k_init holds only workgroups with tiles; a map that does not have the
    // launched shape leaves every row to the solver
    if (*segok_of(a) != 1) return;
    const uint64_t e = reinterpret_cast<const uint64_t*>(a.ws + a.lay.tmap)[blockIdx.x];
    row = (int64_t)(e >> 32);
    part0 = (int64_t)(e & 0xFFFFFFFFu) * K;
  }
  TileCtx c;
  int64_t base;
  row_span(a, row, base, c.d);
  const int64_t rtiles = c.d > kTileElems ? (c.d + kTileElems - 1) / kTileElems : 1;
  if (part0 >= rtiles) return;
  const int nk = (int)min((int64_t)K, rtiles - part0);
  const int64_t t0 = row * a.lay.tiles + part0;  // status word of the first tile
  const RowCtl* ctl = ctl_of(a, row);
  c.row = a.g + base;
  c.lam = ctl->lam;
  c.tcap = ctl->tcap;
  c.live = ctl->done && !(ctl->flags & (GSPAR_FLAG_NONFINITE | GSPAR_FLAG_BADRHO | GSPAR_FLAG_BADSEG | kFlagInternal));
  const uint64_t seed = a.seed_dev ? a.seed_dev[row] : a.seed;
  c.k0 = (uint32_t)seed;
  c.k1 = (uint32_t)(seed >> 32);
  const float inv = ctl->inv_lam;
  const bool fast = c.live && (c.lam == 0.0 || c.lam >= kLamScaledMin);
  const FastCtx fc = fast_ctx(c.lam);
  // a coordinate is capped (p_i = 1) iff |g_i| >= capf, the float with bit pattern tcap, and is then
  // kept whatever its selection test says: nearly always t_i >= 2^32 > x_i, but where the exact
  // criterion was decided by its roundings (a variance budget with eps of about 1e-16) lambda |g_i| may
  // lie anywhere below 1
  float capf, uncapf;  // and the float below it
  memcpy(&capf, &c.tcap, 4);
  const uint32_t below_cap = c.tcap - 1u;
  memcpy(&uncapf, &below_cap, 4);
  uint64_t* st = status_of(a);
  // group j of this lane in a tile is tile group wv * (kWaveElems / 4) + 64 j + lane
  const int tg0 = wv * (kWaveElems / 4) + lane;
  uint64_t agg[K];  // per tile: (capped survivors << 31) | survivors
  // capped-survivor bytes start at zero, so phase 1 writes only the groups that have some
#pragma unroll
  for (int kk = 0; kk < K; ++kk) *reinterpret_cast<uint4*>(&s_capb[kk][16 * tid]) = make_uint4(0u, 0u, 0u, 0u);
  __syncthreads();

#pragma unroll
  for (int kk = 0; kk < K; ++kk) {
    if (kk >= nk) break;
    __builtin_amdgcn_sched_barrier(0);  // keep each tile's loads in its own iteration
    // phase 1 of tile part0 + kk
    const int64_t part = part0 + kk;
    const int64_t q0 = part * (kTileElems / 4) + tg0;
    uint32_t nsel = 0;
    uint32_t run = 0;  // this lane's capped survivors in the tile so far
    float* const capl = &s_capl[kk][wv][lane * kLaneStride];
    // a group's survivors (sel: bit k of byte k), then the values of those that are capped (cz, not 0)
    auto record = [&](int j, const float v[4], uint32_t sel) {
      // the group's code byte: selection bits (0-3) and signs (4-7), the masked bytes summed
      s_code[kk][tg0 + 64 * j] =
          (uint8_t)__builtin_amdgcn_sad_u8(sign_bytes(v, kSignBytes), 0u, __builtin_amdgcn_sad_u8(sel, 0u, 0u));
      nsel += (uint32_t)__popc(sel);
    };
    // top: the group's largest magnitude, the value kept where only one is capped (the sign is in the
    // group's code byte)
    auto capture = [&](int j, const float v[4], float top, uint32_t cz) {
      s_capb[kk][tg0 + 64 * j] = (uint8_t)(cz | (min(run, 15u) << 4));
      if (__builtin_expect((cz & (cz - 1u)) == 0, 1)) {
        capl[min(run, (uint32_t)kLaneCap)] = top;
        ++run;
      } else {
        // every value goes to the next free slot (the row's pad slot once the row is full), and
        // only a capped one takes it, so no lane branches per coordinate
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          capl[min(run, (uint32_t)kLaneCap)] = v[k];
          run += (cz >> k) & 1u;
        }
      }
    };
    auto group = [&](int j, const float4& y) {
      const float v[4] = {y.x, y.y, y.z, y.w};
      uint32_t sel = decide_fast(q0 + 64 * j, v, fc, c.k0, c.k1);
      // capped coordinates are rare: test the group's largest magnitude first
      const float top = max_abs4(v);
      if (top >= capf) {
        float d[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) d[k] = uncapf - fabsf(v[k]);
        const uint32_t capped = sign_bytes(d, kSelBytes);
        sel |= capped;
        capture(j, v, top, __builtin_amdgcn_sad_u8(capped, 0u, 0u));
      }
      record(j, v, sel);
    };
    if (fast && (part + 1) * (int64_t)kTileElems <= c.d) {
      // whole tile inside the row: kSampleBatch unconditional loads in flight per lane
#pragma unroll
      for (int jb = 0; jb < kTileGroups; jb += kSampleBatch) {
        float4 x[kSampleBatch];
#pragma unroll
        for (int u = 0; u < kSampleBatch; ++u) x[u] = load_stream(c.row + 4 * (q0 + 64 * (jb + u)));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < kSampleBatch; ++u) group(jb + u, x[u]);
      }
    } else if (fast && c.d >= 4) {
      // a row's last tile: the same in two batches, coordinates past the row's end as zeros, which are
      // never selected and never capped (16 loads one after another took 4 us more on short rows)
      const int64_t qfull = c.d >> 2;
#pragma unroll 1
      for (int jb = 0; jb < kTileGroups; jb += kSampleBatch) {
        const int64_t qb = q0 + 64 * jb;
        float4 x[kSampleBatch];
        if (4 * (qb - lane) >= c.d) {
          // nothing of the row for this wave: its code bytes all the same
#pragma unroll 1
          for (int u = 0; u < kSampleBatch; ++u) s_code[kk][tg0 + 64 * (jb + u)] = 0;
          continue;
        }
#pragma unroll
        for (int u = 0; u < kSampleBatch; ++u) {
          const int64_t q = qb + 64 * u;
          x[u] = load_stream(c.row + 4 * (q < qfull ? q : qfull - 1));
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < kSampleBatch; ++u) {
          const int64_t q = qb + 64 * u;
          if (q >= qfull) {
            float v[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            if (q == qfull) load4(c.row, q, c.d, v);
            x[u] = make_float4(v[0], v[1], v[2], v[3]);
          }
        }
#pragma unroll
        for (int u = 0; u < kSampleBatch; ++u) group(jb + u, x[u]);
      }
    } else {
#pragma unroll 1
      for (int j = 0; j < kTileGroups; ++j) {
        float v[4];
        uint32_t z = 0, cz = 0;
        // groups past the row's end (the tail of the last tile, and whole tiles past the end of a
        // shorter segment) hold no coordinates
        if (c.live && 4 * (q0 + 64 * j) < c.d) decide_group(c, q0 + 64 * j, v, z, cz);
        else v[0] = v[1] = v[2] = v[3] = 0.0f;
        record(j, v, (z | (z << 8) | (z << 16) | (z << 24)) & kSelBytes);
        if (cz) capture(j, v, max_abs4(v), cz);
      }
    }
    const bool lane_over = run > (uint32_t)kLaneCap;
    uint32_t ncap = run;
    for (int o = 32; o > 0; o >>= 1) {
      nsel += __shfl_xor(nsel, o);
      ncap += __shfl_xor(ncap, o);
    }
    const bool wave_over = __ballot(lane_over) != 0;
    if (lane == 0) {
      s_wsel[kk][wv] = nsel;
      s_wcap[kk][wv] = ncap;
      s_wcl[kk][wv] = wave_over ? 1u : 0u;
    }
    __syncthreads();
    uint32_t tsel = 0, tcp = 0;
    for (int i = 0; i < kTileThreads / 64; ++i) {
      tsel += s_wsel[kk][i];
      tcp += s_wcap[kk][i];
    }
    agg[kk] = ((uint64_t)tcp << 31) | tsel;
    // publish at once: a row's first tile its inclusive prefix, every other tile its aggregate
    if (tid == 0)
      __hip_atomic_store(&st[t0 + kk], (part == 0 ? kStInc : kStAgg) | agg[kk], __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
  }

  // decoupled look-back for the exclusive prefix of the first tile within its row
  if (part0 == 0) {
    if (tid == 0) s_excl = 0;
  } else {
    if (wv == 0) {
      const int64_t t = t0;
      const int64_t first = t - part0;
      int64_t look = t - 1;
      uint64_t ex = 0;
      while (true) {
        const int64_t i = look - lane;
        uint64_t sw = kStInc;
        if (i >= first) sw = __hip_atomic_load(&st[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        // wait only for the predecessors between this tile and the nearest one whose inclusive
        // prefix is published (that boundary can only move closer while waiting)
        uint64_t incl_mask, missing;
        int stop;
        for (int polls = 0;; ++polls) {
          incl_mask = __ballot((sw >> 62) == 2);
          stop = incl_mask ? (__ffsll((unsigned long long)incl_mask) - 1) : 63;
          missing = __ballot((sw >> 62) == 0 && lane <= stop);
          if (!missing || polls == kPolls) break;
          __builtin_amdgcn_s_sleep(4);
          if ((sw >> 62) == 0 && lane <= stop) sw = __hip_atomic_load(&st[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        // predecessors up to `stop` that never published: count them here
        while (missing) {
          const int m = __ffsll((unsigned long long)missing) - 1;
          const uint64_t val = wave_tile_aggregate(c, (look - m) - first, lane);
          if (lane == m) sw = kStAgg | val;
          missing &= missing - 1;
        }
        uint64_t contrib = lane <= stop ? (sw & kStVal) : 0;
        for (int o = 32; o > 0; o >>= 1) contrib += __shfl_xor(contrib, o);
        ex += contrib;
        if (incl_mask) break;
        look -= 64;
      }
      if (lane == 0) {
        s_excl = ex;
        uint64_t run = ex;
        for (int kk = 0; kk < nk; ++kk) {
          run += agg[kk];
          __hip_atomic_store(&st[t0 + kk], kStInc | run, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      }
    }
  }
  if (part0 == 0 && tid == 0) {
    // the row's first workgroup: its later tiles' inclusive prefixes follow from its own aggregates
    uint64_t run = agg[0];
    for (int kk = 1; kk < nk; ++kk) {
      run += agg[kk];
      __hip_atomic_store(&st[t0 + kk], kStInc | run, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  __syncthreads();
  uint64_t excl = s_excl;

  // phase 2, tile by tile: thread tid owns tile groups [16 tid, 16 tid + 16) (bit b of its masks
  // is tile coordinate 64 tid + b)
#pragma unroll
  for (int kk = 0; kk < K; ++kk) {
    if (kk >= nk) break;
    __builtin_amdgcn_sched_barrier(0);
    const int64_t part = part0 + kk;
    uint32_t wbase = 0, wbase_cap = 0;
    for (int i = 0; i < wv; ++i) {
      wbase += s_wsel[kk][i];
      wbase_cap += s_wcap[kk][i];
    }
    const int64_t e0 = part * (int64_t)kTileElems + 64 * tid;
    uint64_t sm = 0, nm = 0, cm = 0;  // selected, negative, capped-and-selected coordinates
    uint32_t cr = 0;                  // hybrid: rank of this thread's first capped survivor in its wave
    uint32_t cwd[4] = {0u, 0u, 0u, 0u};  // this thread's 16 capped-survivor bytes
    if (s_wsel[kk][wv]) {
      const uint4 cw = *reinterpret_cast<const uint4*>(&s_code[kk][16 * tid]);
      uint32_t s0, s1, n0, n1;
      byte_nibbles(cw.x, cw.y, s0, n0);
      byte_nibbles(cw.z, cw.w, s1, n1);
      sm = ((uint64_t)s1 << 32) | s0;
      nm = ((uint64_t)n1 << 32) | n0;
      if (s_wcap[kk][wv]) {
        const uint4 bw = *reinterpret_cast<const uint4*>(&s_capb[kk][16 * tid]);
        cwd[0] = bw.x;
        cwd[1] = bw.y;
        cwd[2] = bw.z;
        cwd[3] = bw.w;
        uint32_t c0, c1, u0, u1;
        byte_nibbles(bw.x, bw.y, c0, u0);
        byte_nibbles(bw.z, bw.w, c1, u1);
        cm = ((uint64_t)c1 << 32) | c0;
        if constexpr (HYB) {
          uint32_t ctot;
          cr = wave_prefix_bits<7>((uint32_t)__popcll(cm), ctot);
        }
      }
      const bool lds_values = s_wcl[kk][wv] == 0;
      // the value of capped survivor b (0..63) of this thread's coordinates: its group 16 tid + b/4
      // was decided by phase-1 lane (16 tid + b/4) mod 64, whose list holds it after the lane's
      // earlier capped survivors (the byte's high nibble) and the group's lower ones
      auto capval = [&](int b) -> float {
        const int gi = b >> 2;
        const uint32_t cb = (cwd[gi >> 2] >> (8 * (gi & 3))) & 0xFFu;
        const uint32_t slot = (cb >> 4) + (uint32_t)__popc(cb & ((1u << (b & 3)) - 1u));
        return signed_as(s_capl[kk][wv][((16 * tid + gi) & 63) * kLaneStride + slot], (uint32_t)(nm >> b) << 31);
      };
      // Staged emission of the wave's n survivors in `mask` (this lane's begin at rank j): kStageEmit at a
      // time, each lane writes its survivors' entries (tile coordinate, 16 bits; value code: sign in bit
      // 15; `more` adds bit 14 and a capped value's place in the LDS rows) at their ranks in
      // the wave's quarter of the code and capped-survivor bytes, which every lane of the wave has read by
      // now (LDS operations of a wave complete in order); then lane l puts out entries l, l + 64, ... so
      // that each store covers consecutive addresses, instead of one address per lane far apart.
      const int32_t t0c = (int32_t)(part * (int64_t)kTileElems);
      // One round (most waves) needs no bound in its loop.
      auto staged = [&](uint64_t mask, uint32_t j, uint32_t n, auto&& more, auto&& put) {
        gs_u16* const si = reinterpret_cast<gs_u16*>(&s_code[kk][wv * (kWaveElems / 4)]);
        gs_u16* const sc = reinterpret_cast<gs_u16*>(&s_capb[kk][wv * (kWaveElems / 4)]);
        uint32_t m0 = (uint32_t)mask, m1 = (uint32_t)(mask >> 32);
        // this lane's survivors of one half of its coordinates
        auto enter = [&](auto bounded, uint32_t& m, uint32_t neg, uint32_t c0, uint32_t w0) {
          while (m) {
            if (decltype(bounded)::value && j - w0 >= (uint32_t)kStageEmit) break;
            const int b = __builtin_ctz(m);
            si[j - w0] = (gs_u16)(c0 + b);
            sc[j - w0] = (gs_u16)(((neg >> b) & 1u) << 15);
            ++j;
            m &= m - 1u;
          }
        };
        const uint32_t n0 = (uint32_t)nm, n1 = (uint32_t)(nm >> 32), c0 = (uint32_t)(64 * tid);
        for (uint32_t w0 = 0; w0 < n; w0 += (uint32_t)kStageEmit) {
          wave_sync();
          if (n <= (uint32_t)kStageEmit) {
            enter(std::false_type{}, m0, n0, c0, 0u);
            enter(std::false_type{}, m1, n1, c0 + 32u, 0u);
          } else {
            enter(std::true_type{}, m0, n0, c0, w0);
            if (!m0) enter(std::true_type{}, m1, n1, c0 + 32u, w0);
          }
          more(sc, w0);
          wave_sync();
          const uint32_t end = min(n - w0, (uint32_t)kStageEmit);
          for (uint32_t i = (uint32_t)lane; i < end; i += 64u) put(w0 + i, si[i], sc[i]);
        }
      };
      if constexpr (!HYB) {
        uint32_t wtot;
        uint64_t pos = (excl & 0x7FFFFFFFull) + wbase + wave_prefix_bits<7>((uint32_t)__popcll(sm), wtot);
        int32_t* __restrict__ oi = a.idx + row * a.cap;
        float* __restrict__ ov = a.val + row * a.cap;
        auto emit = [&](auto from_lds) {
          uint64_t m = sm;
          while (m) {
            const int b = __ffsll((unsigned long long)m) - 1;
            const uint64_t bit = 1ull << b;
            float val = (nm & bit) ? -inv : inv;
            if (cm & bit) {
              if constexpr (decltype(from_lds)::value) val = capval(b);
              else val = c.row[e0 + b];
            }
            if ((int64_t)pos < a.cap) {
              oi[pos] = (int32_t)(e0 + b);
              ov[pos] = val;
            }
            ++pos;
            m &= m - 1;
          }
        };
        const uint64_t wave_end = (excl & 0x7FFFFFFFull) + wbase + s_wsel[kk][wv];
        const uint64_t wpos = (excl & 0x7FFFFFFFull) + wbase;  // the wave's first output slot
        if (lds_values && s_wsel[kk][wv] <= (uint32_t)kDenseEmit && wave_end <= (uint64_t)a.cap &&
            wave_end <= ((uint64_t)1 << 30)) {
          // the common case, staged: every survivor of the wave within the capacity and its capped
          // values in the lanes' LDS rows
          const uint32_t lpre = (uint32_t)(pos - wpos);
          uint64_t mc = cm;
          const float* const capw = &s_capl[kk][wv][0];
          gchar* __restrict__ bi = uniform_ptr(oi) + 4u * (uint32_t)wpos;
          gchar* __restrict__ bv = uniform_ptr(ov) + 4u * (uint32_t)wpos;
          staged(
              sm, lpre, s_wsel[kk][wv],
              [&](gs_u16* sc, uint32_t w0) {
                while (mc) {
                  const int b = __ffsll((unsigned long long)mc) - 1;
                  const uint32_t at = lpre + (uint32_t)__popcll(sm & ((1ull << b) - 1ull)) - w0;
                  if (at >= (uint32_t)kStageEmit) break;
                  const int gi = b >> 2;
                  const uint32_t cb = (cwd[gi >> 2] >> (8 * (gi & 3))) & 0xFFu;
                  const uint32_t slot = (cb >> 4) + (uint32_t)__popc(cb & ((1u << (b & 3)) - 1u));
                  sc[at] = (gs_u16)(0x4000u | ((uint32_t)(nm >> b) << 15) |
                                      (uint32_t)(((16 * tid + gi) & 63) * kLaneStride + slot));
                  mc &= mc - 1;
                }
              },
              [&](uint32_t i, uint32_t x, uint32_t cc) {
                const float cv = capw[cc & 0x3FFu];
                const float val = signed_as((cc & 0x4000u) ? cv : inv, cc << 16);
                GS_STORE_STREAM((GS_GLOBAL(int32_t)*)(bi + 4u * i), t0c + (int32_t)x);
                GS_STORE_STREAM((GS_GLOBAL(float)*)(bv + 4u * i), val);
              });
        } else if (s_wsel[kk][wv] > (uint32_t)kDenseEmit ||
                   (!lds_values && s_wsel[kk][wv] > (uint32_t)kGroupEmit &&
                    s_wcap[kk][wv] > (uint32_t)kGroupCapped)) {
          // many survivors: lane l takes the wave's groups 64 j + l (the order of phase 1 and of
          // this lane's capped-value row), one step j at a time, so the stores of a step fall on a
          // few consecutive lines instead of one line per lane
          const uint64_t base0 = (excl & 0x7FFFFFFFull) + wbase;
          uint32_t carry = 0;
          for (int j = 0; j < kTileGroups; ++j) {
            const int q = wv * (kWaveElems / 4) + 64 * j + lane;  // tile group (decided by this lane)
            const uint32_t code = s_code[kk][q];
            const uint32_t sel = code & 0xFu, neg = code >> 4;
            const uint32_t cb = s_capb[kk][q], cap = cb & sel;
            uint32_t stot;
            const uint32_t sp = wave_prefix_bits<3>((uint32_t)__popc(sel), stot);
            uint64_t p = base0 + carry + sp;
            const int64_t eq = part * (int64_t)kTileElems + 4 * (int64_t)q;
            // one read of the group for all its capped values: a read waits for the stores before it
            float gv[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            if (!lds_values && cap) load4(c.row, eq >> 2, c.d, gv);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              if ((sel >> k) & 1) {
                float val = ((neg >> k) & 1) ? -inv : inv;
                if ((cap >> k) & 1)
                  val = lds_values ? signed_as(s_capl[kk][wv][lane * kLaneStride + (cb >> 4) +
                                                              __popc(cap & ((1u << k) - 1u))], (neg >> k) << 31)
                                   : gv[k];
                if ((int64_t)p < a.cap) {
                  oi[p] = (int32_t)(eq + k);
                  ov[p] = val;
                }
                ++p;
              }
            }
            carry += stot;
          }
        } else if (lds_values) {
          emit(std::true_type{});
        } else {
          emit(std::false_type{});
        }
      } else {
        // hybrid coding (Section 3.3, eqs. 9-10): capped survivors go to Q_A as (index, g_i), the
        // others to Q_B as index | sign << 31 (their value is sign(g_i) / lambda)
        const uint64_t bm = sm & ~cm;
        uint32_t btot;
        const uint64_t excl_cap = (excl >> 31) & 0x7FFFFFFFull;
        uint64_t pa = excl_cap + wbase_cap + cr;
        uint64_t pb = (excl & 0x7FFFFFFFull) - excl_cap + (wbase - wbase_cap) +
                      wave_prefix_bits<7>((uint32_t)__popcll(bm), btot);
        int32_t* __restrict__ oa = a.idx + row * a.cap;
        float* __restrict__ va = a.val + row * a.cap;
        int32_t* __restrict__ ob = a.code_b + row * a.cap_b;
        auto emit_a = [&](auto from_lds) {
          uint64_t m = cm;
          while (m) {
            const int b = __ffsll((unsigned long long)m) - 1;
            float val;
            if constexpr (decltype(from_lds)::value) val = capval(b);
            else val = c.row[e0 + b];
            if ((int64_t)pa < a.cap) {
              oa[pa] = (int32_t)(e0 + b);
              va[pa] = val;
            }
            ++pa;
            m &= m - 1;
          }
        };
        if (s_wsel[kk][wv] > (uint32_t)kDenseEmit) {
          // many survivors: group by group in phase-1 order, as in the compaction above
          uint64_t pa0 = excl_cap + wbase_cap;
          uint64_t pb0 = (excl & 0x7FFFFFFFull) - excl_cap + (wbase - wbase_cap);
          for (int j = 0; j < kTileGroups; ++j) {
            const int q = wv * (kWaveElems / 4) + 64 * j + lane;  // tile group
            const uint32_t code = s_code[kk][q];
            const uint32_t sel = code & 0xFu, neg = code >> 4;
            const uint32_t cb = s_capb[kk][q], cap = cb & sel, oth = sel & ~cap;
            uint32_t atot, btot2;
            uint64_t qa = pa0 + wave_prefix_bits<3>((uint32_t)__popc(cap), atot);
            uint64_t qb = pb0 + wave_prefix_bits<3>((uint32_t)__popc(oth), btot2);
            const int64_t eq = part * (int64_t)kTileElems + 4 * (int64_t)q;
            float gv[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            if (!lds_values && cap) load4(c.row, eq >> 2, c.d, gv);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              if ((cap >> k) & 1) {
                const float val =
                    lds_values ? signed_as(s_capl[kk][wv][lane * kLaneStride + (cb >> 4) +
                                                          __popc(cap & ((1u << k) - 1u))], (neg >> k) << 31)
                               : gv[k];
                if ((int64_t)qa < a.cap) {
                  oa[qa] = (int32_t)(eq + k);
                  va[qa] = val;
                }
                ++qa;
              } else if ((oth >> k) & 1) {
                if ((int64_t)qb < a.cap_b) ob[qb] = (int32_t)((uint32_t)(eq + k) | (((neg >> k) & 1u) << 31));
                ++qb;
              }
            }
            pa0 += atot;
            pb0 += btot2;
          }
        } else {
          if (cm) {
            if (lds_values) emit_a(std::true_type{});
            else emit_a(std::false_type{});
          }
          const uint64_t wpos = (excl & 0x7FFFFFFFull) - excl_cap + (wbase - wbase_cap);
          if (wpos + btot <= (uint64_t)a.cap_b && wpos + btot <= ((uint64_t)1 << 30)) {
            gchar* __restrict__ bo = uniform_ptr(ob) + 4u * (uint32_t)wpos;
            staged(
                bm, (uint32_t)(pb - wpos), btot, [](gs_u16*, uint32_t) {},
                [&](uint32_t i, uint32_t x, uint32_t cc) {
                  GS_STORE_STREAM((GS_GLOBAL(int32_t)*)(bo + 4u * i), (int32_t)((uint32_t)t0c + x + (cc << 16)));
                });
          } else {
            uint64_t m = bm;
            while (m) {
              const int b = __ffsll((unsigned long long)m) - 1;
              if ((int64_t)pb < a.cap_b) ob[pb] = (int32_t)((uint32_t)(e0 + b) | (uint32_t)(((nm >> b) & 1) << 31));
              ++pb;
              m &= m - 1;
            }
          }
        }
      }
    }
    if constexpr (HYB) {
      // dense ternary vector (Section 3.3): 2 on the capped set, sign(g_i) for the other
      // survivors, 0 elsewhere; this thread's 64 coordinates
      if (a.q && e0 < c.d) {
        int8_t* __restrict__ qr = a.q + base + e0;
        uint32_t w[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          uint32_t x = 0;
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const int b = 4 * j + k;
            const uint32_t code = ((cm >> b) & 1) ? 2u : (((sm >> b) & 1) ? (((nm >> b) & 1) ? 0xFFu : 1u) : 0u);
            x |= code << (8 * k);
          }
          w[j] = x;
        }
        if (e0 + 64 <= c.d && ((uintptr_t)qr & 15) == 0) {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            uint4 v;
            v.x = w[4 * j]; v.y = w[4 * j + 1]; v.z = w[4 * j + 2]; v.w = w[4 * j + 3];
            reinterpret_cast<uint4*>(qr)[j] = v;
          }
        } else {
          const int64_t nb = min((int64_t)64, c.d - e0);
          for (int64_t b = 0; b < nb; ++b) qr[b] = (int8_t)((w[b >> 2] >> (8 * (b & 3))) & 0xFF);
        }
      }
    }
    excl += agg[kk];
  }
  if (part0 + nk == rtiles && tid == 0) {
    const uint64_t incl = excl;
    const int64_t n = (int64_t)(incl & 0x7FFFFFFFull);
    const int64_t kc = (int64_t)((incl >> 31) & 0x7FFFFFFFull);
    uint32_t fl = ctl->flags;
    if (!ctl->done) fl |= kFlagInternal;
    if constexpr (!HYB) {
      if (a.nnz) a.nnz[row] = n;
      if (n > a.cap) fl |= GSPAR_FLAG_OVERFLOW;
    } else {
      a.nnz[row] = kc;
      a.nnz_b[row] = n - kc;
      if (a.inv_out) a.inv_out[row] = inv;
      if (kc > a.cap || n - kc > a.cap_b) fl |= GSPAR_FLAG_OVERFLOW;
    }
    if (a.k_out) a.k_out[row] = kc;
    if (a.lam_out) a.lam_out[row] = ctl->lam;
    if (a.flags_out) a.flags_out[row] = fl;
  }
}

// p_i = min(lambda |g_i|, 1), exactly 1 on the capped set. Grid: rows * nb workgroups. Capped
// coordinates are counted per workgroup and added into one of eight per-row lines.
__global__ void __launch_bounds__(256) k_probs(Args a) {
  __shared__ uint32_t s_cnt[4];
  int64_t row, blk;
  if (!hist_block(a, row, blk)) return;
  const RowCtl* ctl = ctl_of(a, row);
  const double lam = ctl->lam;
  const uint32_t tcap = ctl->tcap;
  const bool live =
      ctl->done && !(ctl->flags & (GSPAR_FLAG_NONFINITE | GSPAR_FLAG_BADRHO | GSPAR_FLAG_BADSEG | kFlagInternal));
  int64_t base, len;
  row_span(a, row, base, len);
  const int64_t beg = blk * a.chunk;
  if (beg >= len) return;  // past the end of a shorter segment
  const float* __restrict__ gr = a.g + base;
  float* __restrict__ pr = a.p ? a.p + base : nullptr;
  const int64_t end = min(len, beg + a.chunk);
  uint32_t kc = 0;
  stream_groups<4, 256>(gr, beg, end, [&](int64_t q, const float v[4], uint32_t m) {
    float o[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const uint32_t key = key_of(v[c]);
      const bool capped = live && key != 0 && key >= tcap;
      double pv = capped ? 1.0 : (live ? fmin(lam * (double)fabsf(v[c]), 1.0) : 0.0);
      if (key == 0) pv = 0.0;
      o[c] = (float)pv;
      kc += capped && ((m >> c) & 1);
    }
    if (pr) {
      if (m == 0xF) {
        store_stream(pr + 4 * q, make_float4(o[0], o[1], o[2], o[3]));
      } else {
        for (int c = 0; c < 4; ++c)
          if ((m >> c) & 1) pr[4 * q + c] = o[c];
      }
    }
  });
  for (int o = 32; o > 0; o >>= 1) kc += __shfl_xor(kc, o);
  if ((threadIdx.x & 63) == 0) s_cnt[threadIdx.x >> 6] = kc;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t tot = 0;
    for (int i = 0; i < (int)(blockDim.x / 64); ++i) tot += s_cnt[i];
    if (tot) atomicAdd(&kc_of(a, row)[blk & 7].v, (unsigned long long)tot);
  }
}

// Per-row outputs of the probabilities entry points (one thread per row).
__global__ void __launch_bounds__(64) k_probs_out(Args a) {
  const int64_t row = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (row >= a.rows) return;
  const RowCtl* ctl = ctl_of(a, row);
  const CountLine* kl = kc_of(a, row);
  uint64_t ktot = 0;
  for (int i = 0; i < 8; ++i) ktot += kl[i].v;
  if (a.lam_out) a.lam_out[row] = ctl->lam;
  if (a.k_out) a.k_out[row] = (int64_t)ktot;
  uint32_t fl = ctl->flags;
  if (!ctl->done) fl |= kFlagInternal;
  if (a.flags_out) a.flags_out[row] = fl;
}

// ------------------------------------------------------------------------------------------
// Host side.
// ------------------------------------------------------------------------------------------
// Kernel classes, in the order the instrumented build reports them.
enum KernelClass {
  kcSample = 0, kcStats, kcProbs, kcSolve, kcInit, kcAggregate, kcProbsOut, kcPresample, kcCount
};

#ifdef GSPAR_INSTRUMENT
// Measurement build only: while armed, each launch records a pair of HIP events taken by the
// dispatch itself (hipExtLaunchKernelGGL's start and stop events, the kernel's own execution
// interval), filed under its class.
struct Timing {
  int max = 0;
  int n = 0;
  hipEvent_t* ev = nullptr;
  int* cls = nullptr;
};
static Timing g_timing;
#endif

template <typename... KArgs, typename... Args>
static void launch(int cls, void (*kern)(KArgs...), dim3 grid, dim3 block, hipStream_t s, Args... args) {
#ifdef GSPAR_INSTRUMENT
  if (g_timing.ev && g_timing.n < g_timing.max) {
    const int i = g_timing.n++;
    g_timing.cls[i] = cls;
    hipExtLaunchKernelGGL(kern, grid, block, 0, s, g_timing.ev[2 * i], g_timing.ev[2 * i + 1], 0, args...);
    return;
  }
#endif
  (void)cls;
  hipLaunchKernelGGL(kern, grid, block, 0, s, args...);
}

// a density in [0, 1], or for the variance-budget solver a finite eps >= 0
static bool rho_ok(double rho, int solver = GSPAR_EXACT) {
  return solver == GSPAR_VARIANCE ? (rho >= 0.0 && rho < INFINITY) : (rho >= 0.0 && rho <= 1.0);
}

static int check_common(const float* g, int64_t rows, int64_t d, int64_t ld, int solver, int iters,
                        void* ws, size_t ws_bytes) {
  if (!g || rows < 1 || d < 1 || d > INT32_MAX || ld < d) return GSPAR_ERR_ARG;
  if (solver != GSPAR_GREEDY && solver != GSPAR_EXACT && solver != GSPAR_VARIANCE) return GSPAR_ERR_ARG;
  if (iters < 0 || iters > kMaxIters) return GSPAR_ERR_ARG;
  if (rows > (int64_t)1 << 24) return GSPAR_ERR_ARG;
  const Layout L = layout_of(rows, d, 0);  // the minimum: no candidate buffers
  if ((double)rows * (double)L.tiles >= 2147483647.0) return GSPAR_ERR_ARG;  // sample grid, tickets
  const int64_t min_chunk = d < kMaxChunk ? d : kMaxChunk;
  if ((double)rows * (double)((d + min_chunk - 1) / min_chunk) >= 2147483647.0) return GSPAR_ERR_ARG;
  if (!ws || ((uintptr_t)ws & 255) || ws_bytes < L.total) return GSPAR_ERR_WORKSPACE;
  return GSPAR_OK;
}

static bool rows_aligned(const Args& a);

// Candidate keys per row: the full capacity for rows long enough to predict a band, within what
// the workspace holds beyond its fixed part, on aligned rows of a strided batch with a density
// budget; 0 otherwise.
static int64_t cand_cap_of(const Args& a) {
  if (a.seg || a.solver == GSPAR_VARIANCE || !rows_aligned(a)) return 0;
  const int64_t full = cand_cap_full(a.d);
  if (full == 0) return 0;
  const size_t fixed = layout_of(a.rows, a.d, 0).total;
  if (a.ws_bytes <= fixed) return 0;
  // each key of capacity takes a list slot and a staging slot
  int64_t fit = (int64_t)((a.ws_bytes - fixed) / (2 * sizeof(uint32_t) * (size_t)a.rows));
  fit &= ~(int64_t)63;
  const int64_t cap = fit < full ? fit : full;
  // a workspace that leaves fewer than 2^16 keys (or the full capacity, for shorter rows) runs
  // without a band
  return cap >= (full < (1 << 16) ? full : (1 << 16)) ? cap : 0;
}

static void plan(Args& a) {
  a.lay = layout_of(a.rows, a.d, cand_cap_of(a));
  const int64_t target = 512;
  int64_t chunk;
  if (a.seg) {
    // chosen from the segment lengths so that the nonempty workgroups are resident at once
    chunk = a.seg_chunk;
  } else {
    int64_t nbt = (target + a.rows - 1) / a.rows;
    if (nbt < 1) nbt = 1;
    chunk = (a.d + nbt - 1) / nbt;
  }
  chunk = (chunk + 3) & ~(int64_t)3;
  if (chunk < kMinChunk) chunk = kMinChunk;
  if (chunk > kMaxChunk) chunk = kMaxChunk;
  a.chunk = chunk;
  a.nb = (int)((a.d + chunk - 1) / chunk);
  a.cand_region = (a.lay.cand_cap / a.nb) & ~(int64_t)63;
  if (a.cand_region == 0) a.lay.cand_cap = 0;  // no room for a band
  // the solver's helpers: one for each chunk past a row's first while they can all be resident, else
  // one for every few (at least one for a row of a strided batch)
  const int64_t rest = a.seg ? a.seg_rest : a.rows * (a.nb - 1);
  int64_t step = (rest + kSolveHelpers - 1) / kSolveHelpers;
  if (!a.seg && step > a.nb - 1) step = a.nb - 1;
  a.help_step = step < 1 ? 1 : (int)step;
  a.helpers = (a.nb - 1) / a.help_step;
}

// Every row of a strided batch starts on a 16-byte boundary.
static bool rows_aligned(const Args& a) { return ((uintptr_t)a.g % 16 == 0) && (a.ld % 4 == 0); }

static int launch_solve(Args& a, hipStream_t s) {
  const int64_t zero_items = a.rows * kC1 * (int64_t)(sizeof(Hist1) / 8) + a.rows * a.lay.tiles;
  const bool sq = a.solver == GSPAR_VARIANCE;  // histogram passes that also sum squares
  int ib = (int)((zero_items + 255) / 256);
  if (ib > 1024) ib = 1024;
  if (ib < 1) ib = 1;
  launch(kcInit, k_init, dim3(ib), dim3(256), s, a);
  // rows long enough for a candidate band: a sample of each row predicts it
  const bool cand = a.lay.cand_cap > 0;
  if (cand) launch(kcPresample, k_presample, dim3((unsigned)(a.rows * kPreWG)), dim3(256), s, a);
  // a segmented call launches only the workgroups that hold coordinates (none if every segment
  // is empty)
  const int64_t nblocks = a.seg ? a.seg_blocks : a.rows * a.nb;
  const dim3 grid((unsigned)nblocks);
  if (nblocks > 0) {
    launch(kcStats, sq ? k_stats<true, false> : cand ? k_stats<false, true> : k_stats<false, false>, grid, dim3(kNT),
           s, a);
  }
  const int64_t helpers = a.seg ? a.seg_blocks : a.rows * a.helpers;
  launch(kcSolve,
         sq ? k_solve<GSPAR_VARIANCE> : a.solver == GSPAR_GREEDY ? k_solve<GSPAR_GREEDY> : k_solve<GSPAR_EXACT>,
         dim3((unsigned)(a.rows + helpers)), dim3(kNT), s, a);
  return hipGetLastError() == hipSuccess ? GSPAR_OK : GSPAR_ERR_HIP;
}

template <int K>
static void launch_sample(const Args& a, hipStream_t s) {
  const dim3 grid((unsigned)(a.seg ? a.seg_wgs : a.rows * ((a.lay.tiles + K - 1) / K)));
  launch(kcSample, a.code_b ? k_sample<true, K> : k_sample<false, K>, grid, dim3(kTileThreads), s, a);
}

static int run_sample(Args& a, hipStream_t s) {
  plan(a);
  if ((double)a.rows * (double)a.nb >= 2147483647.0) return GSPAR_ERR_ARG;
  int rc = launch_solve(a, s);
  if (rc) return rc;
  // tiles per workgroup: 1 while every tile can be resident at once, else 2, so that a
  // workgroup's wait for its predecessors' prefix overlaps the decide phase of its second tile
  const int64_t tiles = a.seg ? a.seg_tiles : a.rows * a.lay.tiles;
  if (a.seg ? a.seg_k == 1 : tiles <= kSampleResident) launch_sample<1>(a, s);
  else launch_sample<2>(a, s);
  return hipGetLastError() == hipSuccess ? GSPAR_OK : GSPAR_ERR_HIP;
}

static int run_probs(Args& a, hipStream_t s) {
  plan(a);
  if ((double)a.rows * (double)a.nb >= 2147483647.0) return GSPAR_ERR_ARG;
  int rc = launch_solve(a, s);
  if (rc) return rc;
  const int64_t nblocks = a.seg ? a.seg_blocks : a.rows * a.nb;
  const dim3 grid((unsigned)nblocks);
  if (nblocks > 0) launch(kcProbs, k_probs, grid, dim3(256), s, a);
  launch(kcProbsOut, k_probs_out, dim3((unsigned)((a.rows + 63) / 64)), dim3(64), s, a);
  return hipGetLastError() == hipSuccess ? GSPAR_OK : GSPAR_ERR_HIP;
}

static Args base_args(const float* g, int64_t rows, int64_t d, int64_t ld, int solver, int iters, void* ws,
                      size_t ws_bytes) {
  Args a;
  memset(&a, 0, sizeof(a));
  a.ws_bytes = ws_bytes;
  a.g = g;
  a.rows = rows;
  a.d = d;
  a.ld = ld;
  a.solver = solver;
  a.T = iters;
  a.ws = static_cast<char*>(ws);
  return a;
}

// ------------------------------------------------------------------------------------------
// Aggregation of the workers' sparsified gradients (Algorithm 1, step 6 on one device):
// v_i = (sum over workers m = 0..M-1, in that order, of Q(g^m)_i in fp64) / M, rounded to fp32.
// Input: each worker's ascending (index, value) list as written by the sampling pass.
//
// One workgroup per block of kAggBlock output coordinates, no workspace. For kAggGroup workers at
// a time the workgroup finds where each list enters and leaves its block (a 9-ary search by eight
// lanes per bound, about log_9(n) dependent loads), loads the first kAggThreads entries of every
// one of those ranges at once, then adds them into an fp64 LDS accumulator one worker after
// another (a barrier between workers), so each coordinate's sum is taken in worker order.
// ------------------------------------------------------------------------------------------
constexpr int kAggBlock = 2048;                   // output coordinates per workgroup
constexpr int kAggThreads = 256;
constexpr int kAggLanes = 8;                      // lanes per search
constexpr int kAggGroup = kAggThreads / kAggLanes / 2;  // workers per pass (two searches each)

struct AggArgs {
  const int32_t* idx;
  const float* val;
  int64_t cap;
  const int64_t* nnz;
  int64_t workers, d;
  float* v;
};

__device__ __forceinline__ int64_t agg_len(const AggArgs& a, int64_t m) {
  const int64_t n = a.nnz[m];
  return n < 0 ? 0 : (n < a.cap ? n : a.cap);
}

// Number of entries of id[0, n) below key when the list ascends (its lower bound), found by the
// eight lanes of an aligned lane group: each step probes eight cut points of [lo, hi) and keeps
// the part between the last probe below key and the first one at or above it. For any list the
// result lies in [0, n] and the loop ends, since [lo, hi) shrinks at every step. Every lane of the
// wave must call it (the loop condition is wave-wide).
__device__ int64_t agg_search(const int32_t* id, int64_t n, int64_t key, bool active) {
  const int lane = threadIdx.x & 63, k = lane & (kAggLanes - 1);
  const unsigned long long gmask = 0xFFull << (lane & ~(kAggLanes - 1));
  int64_t lo = 0, hi = active ? n : 0;
  while (__ballot(hi > lo)) {
    const int64_t w = hi - lo;
    const int64_t pk = lo + (w * (k + 1)) / (kAggLanes + 1);
    const bool below = w > 0 && (int64_t)id[pk] < key;
    const int c = __popcll(__ballot(below) & gmask);
    if (w > 0) {
      const int64_t nlo = c == 0 ? lo : lo + (w * c) / (kAggLanes + 1) + 1;
      const int64_t nhi = c == kAggLanes ? hi : lo + (w * (c + 1)) / (kAggLanes + 1);
      hi = nhi;
      lo = nlo < nhi ? nlo : nhi;
    }
  }
  return lo;
}

__global__ void __launch_bounds__(kAggThreads) k_aggregate(AggArgs a) {
  __shared__ double acc[kAggBlock];
  __shared__ int64_t rng[kAggGroup][2];
  const int t = threadIdx.x;
  const int64_t b0 = (int64_t)blockIdx.x * kAggBlock;
  for (int i = t; i < kAggBlock; i += kAggThreads) acc[i] = 0.0;
  for (int64_t m0 = 0; m0 < a.workers; m0 += kAggGroup) {
    const int64_t mg = a.workers - m0 < kAggGroup ? a.workers - m0 : kAggGroup;
    {
      const int q = t / kAggLanes;           // search q: worker m0 + q/2, bound q&1
      const int64_t m = m0 + (q >> 1);
      const bool act = (q >> 1) < mg;
      const int64_t n = act ? agg_len(a, m) : 0;
      const int64_t lb = agg_search(a.idx + (act ? m : 0) * a.cap, n, b0 + (q & 1) * kAggBlock, act);
      if (act && (t & (kAggLanes - 1)) == 0) rng[q >> 1][q & 1] = lb;
    }
    __syncthreads();
    // the first kAggThreads entries of every range, loaded before any is added
    int32_t r[kAggGroup];
    float x[kAggGroup];
#pragma unroll
    for (int k = 0; k < kAggGroup; ++k) {
      r[k] = -1;
      x[k] = 0.0f;
      if (k < mg) {
        const int64_t j = rng[k][0] + t;
        if (j < rng[k][1]) {
          const int64_t rr = (int64_t)a.idx[(m0 + k) * a.cap + j] - b0;
          r[k] = rr >= 0 && rr < kAggBlock ? (int32_t)rr : -1;
          x[k] = a.val[(m0 + k) * a.cap + j];
        }
      }
    }
#pragma unroll
    for (int k = 0; k < kAggGroup; ++k) {
      if (k < mg) {
        if (r[k] >= 0) acc[r[k]] += (double)x[k];
        const int64_t hi = rng[k][1];
        for (int64_t j = rng[k][0] + t + kAggThreads; j < hi; j += kAggThreads) {
          const int64_t rr = (int64_t)a.idx[(m0 + k) * a.cap + j] - b0;
          if (rr >= 0 && rr < kAggBlock) acc[rr] += (double)a.val[(m0 + k) * a.cap + j];
        }
      }
      __syncthreads();
    }
  }
  const double M = (double)a.workers;
  for (int i = t; i < kAggBlock; i += kAggThreads)
    if (b0 + i < a.d) a.v[b0 + i] = (float)(acc[i] / M);
}

// Scratch memory of the no-allocation entry point: one fixed array per GPU, in the code object's
// device memory. Host code never passes the name `scratch` to a kernel (on the host it is only a
// stand-in for the symbol): the array's device address is looked up once per device and kept.
static __device__ __align__(256) unsigned char scratch[GSPAR_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
static void* g_scratch_ptr[kMaxDevices];
static std::mutex g_scratch_mu;

// Device address of the current device's scratch array (nullptr if it cannot be obtained).
static void* scratch_of_current_device() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess) return nullptr;
    g_scratch_ptr[dev] = p;
  }
  return g_scratch_ptr[dev];
}

}  // namespace gspar

using namespace gspar;

#ifdef GSPAR_INSTRUMENT
// ------------------------------------------------------------------------------------------
// Stream probes (measurement build only): the bandwidth a plain kernel reaches on the same
// buffers, to set the path's figures against. Laid out like the statistics pass of one row:
// kProbeGroups workgroups of kNT threads, each streaming one contiguous chunk through the same
// loop (stream_groups, four float4 loads in flight per thread); the read probe adds the values (so
// no load is dead) into one double per wave, the copy probe writes them to dst.
// ------------------------------------------------------------------------------------------
namespace gspar {
constexpr int kProbeGroups = 512;
__global__ void __launch_bounds__(kNT) k_probe_read(const float* __restrict__ src, int64_t n, double* sink) {
  const int64_t chunk = ((n + kProbeGroups - 1) / kProbeGroups + 3) & ~(int64_t)3;
  const int64_t beg = (int64_t)blockIdx.x * chunk, end = min(n, beg + chunk);
  float acc = 0.0f;
  if (beg < end)
    stream_groups<4, kNT>(src, beg, end, [&](int64_t, const float v[4], uint32_t) {
      acc += (v[0] + v[1]) + (v[2] + v[3]);
    });
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
  if ((threadIdx.x & 63) == 0) atomicAdd(sink, (double)acc);
}
__global__ void __launch_bounds__(kNT) k_probe_copy(const float* __restrict__ src, float* __restrict__ dst, int64_t n) {
  const int64_t chunk = ((n + kProbeGroups - 1) / kProbeGroups + 3) & ~(int64_t)3;
  const int64_t beg = (int64_t)blockIdx.x * chunk, end = min(n, beg + chunk);
  if (beg < end)
    stream_groups<4, kNT>(src, beg, end, [&](int64_t q, const float v[4], uint32_t m) {
      if (m == 0xFu) *reinterpret_cast<float4*>(dst + 4 * q) = make_float4(v[0], v[1], v[2], v[3]);
    });
}
}  // namespace gspar
#endif  // GSPAR_INSTRUMENT

extern "C" {

size_t gspar_workspace_bytes(int64_t rows, int64_t d, int solver) {
  if (rows < 1 || d < 1) return 0;
  return layout_of(rows, d, solver == GSPAR_VARIANCE ? 0 : cand_cap_full(d)).total;
}

int64_t gspar_capacity_hint(int64_t d, double rho) {
  if (d < 1 || !rho_ok(rho)) return 0;
  const double B = rho * (double)d;
  double c = std::ceil(B + 8.0 * std::sqrt(B) + 64.0);
  if (c > (double)d) c = (double)d;
  return (int64_t)c;
}

int sparsify_probs(const float* g, int64_t d, double rho, int solver, int greedy_iters, float* p,
                   double* lambda, int64_t* k, uint32_t* flags, void* ws, size_t ws_bytes, void* stream) {
  if (!lambda || !rho_ok(rho, solver)) return GSPAR_ERR_ARG;
  int rc = check_common(g, 1, d, d, solver, greedy_iters, ws, ws_bytes);
  if (rc) return rc;
  Args a = base_args(g, 1, d, d, solver, greedy_iters, ws, ws_bytes);
  a.rho = rho;
  a.p = p;
  a.lam_out = lambda;
  a.k_out = k;
  a.flags_out = flags;
  return run_probs(a, (hipStream_t)stream);
}

int sparsify_sample_compact(const float* g, int64_t d, double rho, int solver, int greedy_iters, uint64_t seed,
                            int32_t* idx, float* val, int64_t capacity, int64_t* nnz, double* lambda, int64_t* k,
                            uint32_t* flags, void* ws, size_t ws_bytes, void* stream) {
  if (!nnz || capacity < 0 || (capacity > 0 && (!idx || !val)) || !rho_ok(rho, solver)) return GSPAR_ERR_ARG;
  int rc = check_common(g, 1, d, d, solver, greedy_iters, ws, ws_bytes);
  if (rc) return rc;
  Args a = base_args(g, 1, d, d, solver, greedy_iters, ws, ws_bytes);
  a.rho = rho;
  a.seed = seed;
  a.idx = idx;
  a.val = val;
  a.cap = capacity;
  a.nnz = nnz;
  a.lam_out = lambda;
  a.k_out = k;
  a.flags_out = flags;
  return run_sample(a, (hipStream_t)stream);
}

int sparsify_sample_hybrid_batched(const float* g, int64_t rows, int64_t d, int64_t ld, const double* rho,
                                   int solver, int greedy_iters, const uint64_t* seeds, int32_t* idx_a, float* val_a,
                                   int64_t cap_a, int64_t* n_a, int32_t* code_b, int64_t cap_b, int64_t* n_b,
                                   float* inv_lambda, int8_t* q, double* lambda, uint32_t* flags, void* ws,
                                   size_t ws_bytes, void* stream) {
  if (!rho || !seeds || !n_a || !n_b || cap_a < 0 || cap_b < 0 || (cap_a > 0 && (!idx_a || !val_a)) ||
      !code_b)
    return GSPAR_ERR_ARG;
  int rc = check_common(g, rows, d, ld, solver, greedy_iters, ws, ws_bytes);
  if (rc) return rc;
  Args a = base_args(g, rows, d, ld, solver, greedy_iters, ws, ws_bytes);
  a.rho_dev = rho;
  a.seed_dev = seeds;
  a.idx = idx_a;
  a.val = val_a;
  a.cap = cap_a;
  a.nnz = n_a;
  a.code_b = code_b;
  a.cap_b = cap_b;
  a.nnz_b = n_b;
  a.inv_out = inv_lambda;
  a.q = q;
  a.lam_out = lambda;
  a.flags_out = flags;
  return run_sample(a, (hipStream_t)stream);
}

int sparsify_sample_hybrid(const float* g, int64_t d, double rho, int solver, int greedy_iters, uint64_t seed,
                           int32_t* idx_a, float* val_a, int64_t cap_a, int64_t* n_a, int32_t* code_b, int64_t cap_b,
                           int64_t* n_b, float* inv_lambda, int8_t* q, double* lambda, uint32_t* flags, void* ws,
                           size_t ws_bytes, void* stream) {
  if (!n_a || !n_b || cap_a < 0 || cap_b < 0 || (cap_a > 0 && (!idx_a || !val_a)) || !code_b ||
      !rho_ok(rho, solver))
    return GSPAR_ERR_ARG;
  int rc = check_common(g, 1, d, d, solver, greedy_iters, ws, ws_bytes);
  if (rc) return rc;
  Args a = base_args(g, 1, d, d, solver, greedy_iters, ws, ws_bytes);
  a.rho = rho;
  a.seed = seed;
  a.idx = idx_a;
  a.val = val_a;
  a.cap = cap_a;
  a.nnz = n_a;
  a.code_b = code_b;
  a.cap_b = cap_b;
  a.nnz_b = n_b;
  a.inv_out = inv_lambda;
  a.q = q;
  a.lam_out = lambda;
  a.flags_out = flags;
  return run_sample(a, (hipStream_t)stream);
}

int gspar_coding_bits(int64_t d, int64_t n_a, int64_t n_b, int64_t n_b_neg, int float_bits, double* out) {
  if (!out || d < 1 || n_a < 0 || n_b < 0 || n_b_neg < 0 || n_b_neg > n_b || n_a > d || n_b > d - n_a ||
      float_bits < 1)
    return GSPAR_ERR_ARG;
  const double L = std::log2((double)d), b = (double)float_bits;
  // Q_A: index and value per entry; Q_B: index and sign per entry; one float for 1/lambda
  out[0] = (double)n_a * (b + L) + (double)n_b * (L + 1.0) + b;
  // entropy-coded ternary vector (symbols 2, -1, +1, 0) plus the values of Q_A and 1/lambda
  const double counts[4] = {(double)n_a, (double)n_b_neg, (double)(n_b - n_b_neg), (double)(d - n_a - n_b)};
  double h = 0.0;
  for (double c : counts)
    if (c > 0.0) h += c * std::log2((double)d / c);
  out[1] = h + (double)n_a * b + b;
  // the experiments' per-message cost, with the realised |Q_B| for the expected sum of p over it
  out[2] = (double)n_a * (b + L) + std::min(2.0 * (double)d, (double)n_b * L) + b;
  return GSPAR_OK;
}

int gspar_aggregate(const int32_t* idx, const float* val, int64_t cap, const int64_t* nnz, int64_t workers, int64_t d,
                    float* v, void* stream) {
  using namespace gspar;
  if (!nnz || !v || workers < 1 || workers > ((int64_t)1 << 20) || d < 1 || d > INT32_MAX || cap < 0 ||
      (cap > 0 && (!idx || !val)))
    return GSPAR_ERR_ARG;
  AggArgs a;
  a.idx = idx;
  a.val = val;
  a.cap = cap;
  a.nnz = nnz;
  a.workers = workers;
  a.d = d;
  a.v = v;
  hipStream_t s = (hipStream_t)stream;
  launch(kcAggregate, k_aggregate, dim3((unsigned)((d + kAggBlock - 1) / kAggBlock)), dim3(kAggThreads), s, a);
  return hipGetLastError() == hipSuccess ? GSPAR_OK : GSPAR_ERR_HIP;
}

int sparsify_probs_batched(const float* g, int64_t rows, int64_t d, int64_t ld, const double* rho, int solver,
                           int greedy_iters, float* p, double* lambda, int64_t* k, uint32_t* flags, void* ws,
                           size_t ws_bytes, void* stream) {
  if (!rho || !lambda) return GSPAR_ERR_ARG;
  int rc = check_common(g, rows, d, ld, solver, greedy_iters, ws, ws_bytes);
  if (rc) return rc;
  Args a = base_args(g, rows, d, ld, solver, greedy_iters, ws, ws_bytes);
  a.rho_dev = rho;
  a.p = p;
  a.lam_out = lambda;
  a.k_out = k;
  a.flags_out = flags;
  return run_probs(a, (hipStream_t)stream);
}

int sparsify_sample_compact_batched(const float* g, int64_t rows, int64_t d, int64_t ld, const double* rho,
                                    int solver, int greedy_iters, const uint64_t* seeds, int32_t* idx, float* val,
                                    int64_t cap_per_row, int64_t* nnz, double* lambda, int64_t* k, uint32_t* flags,
                                    void* ws, size_t ws_bytes, void* stream) {
  if (!rho || !seeds || !nnz || cap_per_row < 0 || (cap_per_row > 0 && (!idx || !val))) return GSPAR_ERR_ARG;
  int rc = check_common(g, rows, d, ld, solver, greedy_iters, ws, ws_bytes);
  if (rc) return rc;
  Args a = base_args(g, rows, d, ld, solver, greedy_iters, ws, ws_bytes);
  a.rho_dev = rho;
  a.seed_dev = seeds;
  a.idx = idx;
  a.val = val;
  a.cap = cap_per_row;
  a.nnz = nnz;
  a.lam_out = lambda;
  a.k_out = k;
  a.flags_out = flags;
  return run_sample(a, (hipStream_t)stream);
}

int sparsify_sample_compact_batched_noalloc(const float* g, int64_t rows, int64_t d, int64_t ld, const double* rho,
                                            int solver, int greedy_iters, const uint64_t* seeds, int32_t* idx,
                                            float* val, int64_t cap_per_row, int64_t* nnz, double* lambda, int64_t* k,
                                            uint32_t* flags, void* stream) {
  if (rows < 1 || d < 1) return GSPAR_ERR_ARG;
  if (layout_of(rows, d, 0).total > GSPAR_SCRATCH_BYTES) return GSPAR_ERR_TOO_LARGE;
  void* ws = scratch_of_current_device();
  if (!ws) return GSPAR_ERR_HIP;
  return sparsify_sample_compact_batched(g, rows, d, ld, rho, solver, greedy_iters, seeds, idx, val, cap_per_row,
                                         nnz, lambda, k, flags, ws, GSPAR_SCRATCH_BYTES, stream);
}

// Host check of segment offsets (off[0] >= 0, nondecreasing, every length below 2^31): the longest
// length (at least 1, the row length the workspace is sized for), the total length, and whether
// every segment is aligned (g 16-byte aligned and every start a multiple of 4).
static int check_segments(const float* g, const int64_t* off, const int64_t* off_dev, int64_t segs, int64_t& maxlen,
                          int64_t& total, bool& aligned) {
  if (!g || !off || !off_dev || segs < 1 || segs > ((int64_t)1 << 24) || off[0] < 0) return GSPAR_ERR_ARG;
  maxlen = 1;
  aligned = (uintptr_t)g % 16 == 0;
  for (int64_t r = 0; r < segs; ++r) {
    const int64_t len = off[r + 1] - off[r];
    if (off[r + 1] < off[r] || len > INT32_MAX) return GSPAR_ERR_ARG;
    if (len > maxlen) maxlen = len;
    if (off[r] & 3) aligned = false;
  }
  total = off[segs] - off[0];
  return GSPAR_OK;
}

static void set_segments(Args& a, const int64_t* off, const int64_t* off_dev, int64_t segs, int64_t total,
                         bool aligned) {
  a.seg = off_dev;
  a.seg_total = off[segs];
  a.seg_elems = total;
  a.seg_align = aligned ? 1 : 0;
  // histogram passes: the smallest chunk (a multiple of 4, at least kMinChunk) for which the
  // segments need at most 512 workgroups (two resident per CU); the grid holds exactly those
  auto blocks = [&](int64_t ch) {
    int64_t n = 0;
    for (int64_t r = 0; r < segs; ++r) n += (off[r + 1] - off[r] + ch - 1) / ch;
    return n;
  };
  int64_t lo = kMinChunk, hi = kMaxChunk & ~(int64_t)3;
  if (blocks(lo) <= 512) {
    hi = lo;
  } else if (blocks(hi) <= 512) {
    while (hi - lo > 4) {
      const int64_t mid = ((lo + hi) / 2) & ~(int64_t)3;
      if (blocks(mid) <= 512) hi = mid;
      else lo = mid;
    }
  }
  a.seg_chunk = hi;
  a.seg_blocks = blocks(hi);
  a.seg_rest = a.seg_blocks;
  for (int64_t r = 0; r < segs; ++r) a.seg_rest -= off[r + 1] > off[r];
  // sample pass: tiles per workgroup from the tiles that hold coordinates, and the workgroups
  a.seg_tiles = 0;
  for (int64_t r = 0; r < segs; ++r) {
    const int64_t len = off[r + 1] - off[r];
    a.seg_tiles += len > kTileElems ? (len + kTileElems - 1) / kTileElems : 1;
  }
  a.seg_k = a.seg_tiles <= kSampleResident ? 1 : 2;
  a.seg_wgs = 0;
  for (int64_t r = 0; r < segs; ++r) {
    const int64_t len = off[r + 1] - off[r];
    const int64_t rt = len > kTileElems ? (len + kTileElems - 1) / kTileElems : 1;
    a.seg_wgs += (rt + a.seg_k - 1) / a.seg_k;
  }
}

int sparsify_sample_compact_segmented(const float* g, int64_t segs, const int64_t* off, const int64_t* off_dev,
                                      const double* rho, int solver, int greedy_iters, const uint64_t* seeds,
                                      int32_t* idx, float* val, int64_t cap_per_seg, int64_t* nnz, double* lambda,
                                      int64_t* k, uint32_t* flags, void* ws, size_t ws_bytes, void* stream) {
  if (!rho || !seeds || !nnz || cap_per_seg < 0 || (cap_per_seg > 0 && (!idx || !val))) return GSPAR_ERR_ARG;
  int64_t maxlen, total;
  bool aligned;
  int rc = check_segments(g, off, off_dev, segs, maxlen, total, aligned);
  if (rc) return rc;
  rc = check_common(g, segs, maxlen, maxlen, solver, greedy_iters, ws, ws_bytes);
  if (rc) return rc;
  Args a = base_args(g, segs, maxlen, maxlen, solver, greedy_iters, ws, ws_bytes);
  set_segments(a, off, off_dev, segs, total, aligned);
  a.rho_dev = rho;
  a.seed_dev = seeds;
  a.idx = idx;
  a.val = val;
  a.cap = cap_per_seg;
  a.nnz = nnz;
  a.lam_out = lambda;
  a.k_out = k;
  a.flags_out = flags;
  return run_sample(a, (hipStream_t)stream);
}

int sparsify_sample_hybrid_segmented(const float* g, int64_t segs, const int64_t* off, const int64_t* off_dev,
                                     const double* rho, int solver, int greedy_iters, const uint64_t* seeds,
                                     int32_t* idx_a, float* val_a, int64_t cap_a, int64_t* n_a, int32_t* code_b,
                                     int64_t cap_b, int64_t* n_b, float* inv_lambda, int8_t* q, double* lambda,
                                     uint32_t* flags, void* ws, size_t ws_bytes, void* stream) {
  if (!rho || !seeds || !n_a || !n_b || cap_a < 0 || cap_b < 0 || (cap_a > 0 && (!idx_a || !val_a)) ||
      !code_b)
    return GSPAR_ERR_ARG;
  int64_t maxlen, total;
  bool aligned;
  int rc = check_segments(g, off, off_dev, segs, maxlen, total, aligned);
  if (rc) return rc;
  rc = check_common(g, segs, maxlen, maxlen, solver, greedy_iters, ws, ws_bytes);
  if (rc) return rc;
  Args a = base_args(g, segs, maxlen, maxlen, solver, greedy_iters, ws, ws_bytes);
  set_segments(a, off, off_dev, segs, total, aligned);
  a.rho_dev = rho;
  a.seed_dev = seeds;
  a.idx = idx_a;
  a.val = val_a;
  a.cap = cap_a;
  a.nnz = n_a;
  a.code_b = code_b;
  a.cap_b = cap_b;
  a.nnz_b = n_b;
  a.inv_out = inv_lambda;
  a.q = q;
  a.lam_out = lambda;
  a.flags_out = flags;
  return run_sample(a, (hipStream_t)stream);
}

int sparsify_probs_segmented(const float* g, int64_t segs, const int64_t* off, const int64_t* off_dev,
                             const double* rho, int solver, int greedy_iters, float* p, double* lambda, int64_t* k,
                             uint32_t* flags, void* ws, size_t ws_bytes, void* stream) {
  if (!rho || !lambda) return GSPAR_ERR_ARG;
  int64_t maxlen, total;
  bool aligned;
  int rc = check_segments(g, off, off_dev, segs, maxlen, total, aligned);
  if (rc) return rc;
  rc = check_common(g, segs, maxlen, maxlen, solver, greedy_iters, ws, ws_bytes);
  if (rc) return rc;
  Args a = base_args(g, segs, maxlen, maxlen, solver, greedy_iters, ws, ws_bytes);
  set_segments(a, off, off_dev, segs, total, aligned);
  a.rho_dev = rho;
  a.p = p;
  a.lam_out = lambda;
  a.k_out = k;
  a.flags_out = flags;
  return run_probs(a, (hipStream_t)stream);
}

const char* gspar_status_string(int status) {
  switch (status) {
    case GSPAR_OK: return "ok";
    case GSPAR_ERR_ARG: return "invalid argument";
    case GSPAR_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case GSPAR_ERR_HIP: return "HIP launch failed";
    case GSPAR_ERR_TOO_LARGE: return "problem too large for the library's fixed scratch array";
    default: return "unknown status";
  }
}

int gspar_version(void) { return 100; }

#ifdef GSPAR_INSTRUMENT
int gspar_prof_arm(int max_launches) {
  if (max_launches < 1) return GSPAR_ERR_ARG;
  gspar_prof_disarm();
  g_timing.ev = new hipEvent_t[2 * (size_t)max_launches];
  g_timing.cls = new int[(size_t)max_launches];
  for (int i = 0; i < 2 * max_launches; ++i) {
    if (hipEventCreate(&g_timing.ev[i]) != hipSuccess) {
      for (int j = 0; j < i; ++j) (void)hipEventDestroy(g_timing.ev[j]);
      delete[] g_timing.ev;
      delete[] g_timing.cls;
      g_timing = Timing();
      return GSPAR_ERR_HIP;
    }
  }
  g_timing.max = max_launches;
  g_timing.n = 0;
  return GSPAR_OK;
}

int gspar_prof_read(double* ms, int* launches) {
  if (!ms || !launches) return GSPAR_ERR_ARG;
  for (int c = 0; c < kcCount; ++c) {
    ms[c] = 0.0;
    launches[c] = 0;
  }
  if (!g_timing.ev || g_timing.n == 0) return GSPAR_OK;
  if (hipEventSynchronize(g_timing.ev[2 * g_timing.n - 1]) != hipSuccess) return GSPAR_ERR_HIP;
  for (int i = 0; i < g_timing.n; ++i) {
    float t = 0.f;
    if (hipEventElapsedTime(&t, g_timing.ev[2 * i], g_timing.ev[2 * i + 1]) != hipSuccess) return GSPAR_ERR_HIP;
    ms[g_timing.cls[i]] += t;
    launches[g_timing.cls[i]] += 1;
  }
  return GSPAR_OK;
}

int gspar_prof_disarm(void) {
  if (g_timing.ev) {
    for (int i = 0; i < 2 * g_timing.max; ++i) (void)hipEventDestroy(g_timing.ev[i]);
    delete[] g_timing.ev;
    delete[] g_timing.cls;
  }
  g_timing = Timing();
  return GSPAR_OK;
}

// Host-side checks of the device arithmetic (the same source compiled for the host): rounding of
// the exact sums, the shift invariant, the capped-threshold search and the generator.
double gspar_check_fx_round(const uint64_t* limbs5) {
  uint64_t d[kDig] = {};
  for (int i = 0; i < 5; ++i) {
    d[2 * i] += limbs5[i] & 0xFFFFFFFFull;
    d[2 * i + 1] += limbs5[i] >> 32;
  }
  return dig_round<kDig>(d, -149);
}

// v * 2^s added to digits, then carried into 64-bit limbs.
static uint32_t check_digits(uint64_t v, int s, int smax, uint64_t* d) {
  int at;
  uint64_t x[3];
  const uint32_t err = dig_split(v, s, smax, at, x);
  for (int i = 0; i < 3; ++i) d[at + i] += x[i];
  return err;
}
static void check_limbs(uint64_t* d, int limbs, uint64_t* out) {
  uint64_t carry = 0;
  for (int i = 0; i < 2 * limbs; ++i) {
    const uint64_t v = d[i] + carry;
    carry = v >> 32;
    if (i & 1) out[i / 2] |= v << 32;
    else out[i / 2] = v & 0xFFFFFFFFull;
  }
}

uint32_t gspar_check_fx_shifted(uint64_t v, int s, uint64_t* limbs5) {
  uint64_t d[kDig] = {};
  const uint32_t err = check_digits(v, s, 255, d);
  check_limbs(d, 5, limbs5);
  return err;
}

uint32_t gspar_check_fq_squares(uint64_t qh, uint64_t ql, int shift, uint64_t* limbs10) {
  uint64_t d[kDigSq] = {};
  uint32_t err = kFlagInternal;
  if (shift >= 0 && shift <= 255)
    err = check_digits(qh, 2 * shift + 24, 2 * 255 + 24, d) | check_digits(ql, 2 * shift, 2 * 255, d);
  check_limbs(d, 10, limbs10);
  return err;
}

double gspar_check_exact_sum(const float* x, int64_t n) {
  uint64_t d[kDig] = {};
  uint32_t err = 0;
  for (int64_t i = 0; i < n; ++i) {
    const uint32_t key = key_of(x[i]);
    if (key == 0 || key >= kKeyInf) continue;
    err |= check_digits(key_sig(key), binade_shift((int)(key >> 23)), 255, d);
  }
  return err ? NAN : dig_round<kDig>(d, -149);
}

uint32_t gspar_check_cap_key(double lam) { return cap_key(lam); }

int gspar_probe_stream(const float* src, float* dst, int64_t n, double* sink, void* stream) {
  if (!src || n < 0 || n % 4 != 0 || (uintptr_t)src % 16 || (dst && (uintptr_t)dst % 16) || (!dst && !sink))
    return GSPAR_ERR_ARG;
  if (n == 0) return GSPAR_OK;
  hipStream_t s = (hipStream_t)stream;
  const dim3 grid(kProbeGroups), block(kNT);
  if (dst) hipLaunchKernelGGL(k_probe_copy, grid, block, 0, s, src, dst, n);
  else hipLaunchKernelGGL(k_probe_read, grid, block, 0, s, src, n, sink);
  return hipGetLastError() == hipSuccess ? GSPAR_OK : GSPAR_ERR_HIP;
}

void gspar_check_philox(const uint32_t* ctr, const uint32_t* key, uint32_t* out) {
  uint32_t c0 = ctr[0], c1 = ctr[1], c2 = ctr[2], c3 = ctr[3];
  philox10(c0, c1, c2, c3, key[0], key[1]);
  out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}
#endif  // GSPAR_INSTRUMENT

}  // extern "C"
