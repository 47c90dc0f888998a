// Device decoder for container format v2 on gfx950 (CDNA4, wave64).
//
// One workgroup of 256 threads (4 waves) decodes one 16 KiB block at a time
// into an LDS tile:
//   0. the block's payload prefix is copied into LDS and the four stream
//      headers are parsed from that copy;
//   1. three waves decode the command (CMD), match-length (MLEN) and offset
//      (OFF) streams, one each, reading their rANS words from the LDS copy;
//   2. one block-wide scan turns literal-run and match lengths into literal
//      and output positions (command placement), counts the matches whose
//      source touches the block itself in sequence order, and lists the
//      matches whose source lies wholly in earlier blocks;
//   3. the literal stream's 64-lane groups are decoded by one wave each, every
//      literal written straight to its output position in the tile; then the
//      matches from earlier blocks are copied from HBM;
//   4. the matches whose source touches the block are resolved in dependency
//      passes by wave 0: a match is copied once every earlier match that
//      writes into its source window is done; byte-sequential overlap is
//      unrolled by period.  Meanwhile waves 1..3 do stages 0 and 1 of the
//      workgroup's next block (its payload prefix goes into the literal
//      rings, idle until the next literal stage);
//   5. the tile is written to HBM with 16-byte stores.
// Blocks are taken in dependency-level order ("wavefront" order, paper:
// Background section).  One launch decodes them all: a workgroup takes its
// blocks by ticket, does everything of a block that needs no other block, and
// waits for the completion flags of the blocks it copies from only before
// those copies.  (Static slices, of one level or of each level in a launch of
// its own, are the other mode.)
// No MFMA: nothing here is a contraction.
#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "lz_device.h"
#include "lz_internal.h"

namespace {

constexpr uint32_t kWG = 256;
constexpr uint32_t kWaves = kWG / 64;
constexpr uint32_t kB = 1u << kMaxBlockLog2;      // largest block: 16 KiB tile
constexpr uint32_t kMaxSeq = 1025;                // B/m + 1 for B = 16 KiB, m = 16
constexpr uint32_t kLutLit = 1u << kMaxPLit;      // 4096 packed literal entries
constexpr uint32_t kL = 1u << 16;                 // rANS state lower bound
constexpr uint32_t kFastLen = 256;                // longest in-block match copied in pieces
constexpr uint32_t kClkSlots = 16;                // stage clocks: 9 stages, block count, events
constexpr uint32_t kPrepRing = 5120;              // payload prefix kept in the literal rings
constexpr uint32_t kBuckets = 128;                // a short stream's slots in so many buckets
constexpr uint32_t kDeps = 256;                   // dependencies whose ids are kept in LDS

// Stage clocks (instrumented build only, -DLZ_STAGE_CLOCKS): a barrier, then
// thread 0 adds the cycles since the previous mark to stage i.  The product
// build compiles these to nothing.
#ifdef LZ_STAGE_CLOCKS
#define CLK_START(S) do { if (threadIdx.x == 0) (S).clk_last = __builtin_readcyclecounter(); } while (0)
#define CLK_MARK(S, i)                                          \
  do {                                                          \
    __syncthreads();                                            \
    if (threadIdx.x == 0) {                                     \
      const uint64_t c_ = __builtin_readcyclecounter();         \
      (S).clk[i] += c_ - (S).clk_last;                          \
      (S).clk_last = c_;                                        \
    }                                                           \
  } while (0)
// event counters (slots 10..15): CLK_ADD(S, i, v) by lane 0 of wave 0
#define CLK_ADD(S, i, v) do { if (threadIdx.x == 0) (S).clk[i] += (v); } while (0)
// the same for lane 0 of wave 1
#define CLK_ADD1(S, i, v) do { if (threadIdx.x == 64) (S).clk[i] += (v); } while (0)
#define CLK_NOW() __builtin_readcyclecounter()
#else
#define CLK_START(S) do { } while (0)
#define CLK_MARK(S, i) do { } while (0)
#define CLK_ADD(S, i, v) do { } while (0)
#define CLK_ADD1(S, i, v) do { } while (0)
#define CLK_NOW() 0ull
#endif

// All LDS is static: 53,728 B.  Three workgroups per CU need at most 53,760 B
// each (LDS is handed out in pieces of 1,280 B, 128 per CU).
struct Smem {
  uint32_t lut[kLutLit];       // literal decode entries: symbol | f << 8 | (slot - c) << 20
  // right after the table, so that one index reaches both: an entry's index is
  // its slot, or kLutLit + 256 wave + place in the ring
  union {
    struct {
      uint32_t ringe[kWaves][256]; // rANS words of the literal stream staged per wave:
      uint16_t ring[kWaves][256];  // the table entry of a word's slot, and the word
    };
    struct {                       // between literal stages:
      alignas(16) uint8_t prep[kPrepRing];   // the next block's payload prefix (prep_ring)
      uint32_t dep[kDeps];                   // the blocks it copies from
    };
  };
  alignas(16) uint8_t tile[kB + 16];   // output tile (16-byte reads may start at its last
                               // byte); until stage 3 a copy of the payload prefix
  // CMD, MLEN, OFF: the symbols that occur, in order (the k-th one: its first
  // slot and its value), and which of them owns the first slot of each bucket
  uint16_t cum[3][257];
  uint8_t sym[3][256];
  uint8_t bkt[3][kBuckets];
  uint16_t lit[kMaxSeq + 1];   // LL, then literal start of each sequence ([ns] = n_lit);
                               // stage 4: destination of in-block match a
  uint16_t out[kMaxSeq + 1];   // ML, then output start of each sequence ([ns] = block length);
                               // stage 4: length of in-block match a
  uint32_t oflo[kMaxSeq];      // absolute source offsets, low 32 bits; stage 4: packed
                               // source, period and dependency flag of in-block match a
  uint8_t ofhi[kMaxSeq + 3];   // offset bits 32..39
  uint16_t lst[kMaxSeq];       // [0, n_ext): matches from earlier blocks (any order);
                               // [kMaxSeq - n_in, kMaxSeq): in-block matches, last first;
                               // stage 4: dependency range of in-block match a
  union {
    struct {
      uint16_t fdst[64], flen[64], frng[64]; // at most 64 in-block matches: destination,
      uint32_t fpk[64];                      // length, dependency range, source | period
    };
    uint64_t rdy[64];          // once those are in registers: the matches a pass copies
  };                           // (destination | length << 16 | source << 32)
  uint32_t pst[7];             // literal record of the prepared block
  uint32_t pdir[4];            // its payload offset (low, high word), sequences, literals
  uint32_t plw[kWaves], pln[kWaves];   // its literal groups' first words and word counts
  uint32_t pok;                // prepared block: records valid
  uint32_t scan[3][kWaves];
  uint32_t perr[3];            // prepared block: short stream k failed its checks
  uint32_t ndep, wait, used;   // prepared block: how many blocks it copies from; not all done
                               // yet; some block copies from it
  uint32_t err, next, nin;
  uint32_t nit, nb;            // the workgroup's next ticket and block
#ifdef LZ_STAGE_CLOCKS
  uint64_t clk[kClkSlots], clk_last;
#endif
};

static_assert(offsetof(Smem, ringe) == 4 * kLutLit && kLutLit % 1024 == 0, "one index for table and rings");

struct DevArgs {
  const uint8_t* arc;
  uint64_t n, off_tables, off_dir, off_dep_ptr, off_dep_idx, off_payload;
  uint32_t bl, w, m, lit_lanes, seq_lanes;
  uint32_t P[4];
  const uint32_t* lut;      // workspace literal LUT image
  const uint32_t* queue;    // block ids in level order
  const uint32_t* qptr;     // request mode: device slice bounds (q_begin/q_end index it)
  uint32_t q_begin, q_end;  // static slice of the queue
  uint8_t* out;             // whole-file output base (direct mode)
  const uint64_t* addr;     // request mode: per-block device address, or null
  uint32_t* flags;          // per block: the epoch it was last decoded in
  uint32_t* ctl;
  uint32_t wg0, nwg;        // the launch's workgroups wg0 .. wg0 + nwg - 1 decode this archive
  uint32_t flow;            // 1, 2: blocks by ticket, ordered by completion flags (2: blocks
                            // share cache lines of the output)
  uint32_t spin_limit;
};

__device__ __forceinline__ uint32_t lane_id() { return threadIdx.x & 63; }
// 16 bytes per lane straight from global memory into LDS, without registers
// (global_load_lds_dwordx4): lane k's bytes land at dst + 16 k, dst being the
// wave's uniform LDS address.  The compiler does not track the LDS write:
// vm_wait() (vmcnt(0)) must come before any read of the bytes.
__device__ __forceinline__ void lds_dma16(const void* src, void* dst) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                   (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
}
__device__ __forceinline__ void vm_wait() {
  __builtin_amdgcn_s_waitcnt(0xF70);   // vmcnt(0), expcnt and lgkmcnt untouched
}
// This wave's stores have completed: what a flag says that is set afterwards.
// The wait alone is no order to the compiler, which may move relaxed stores
// across it; the fences are (they cost no instruction here).
__device__ __forceinline__ void stores_done() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  vm_wait();
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
}
__device__ __forceinline__ uint32_t uni(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }

__device__ __forceinline__ uint32_t mbcnt(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

__device__ __forceinline__ void latch(uint32_t* ctl, uint32_t bits) {
  __hip_atomic_fetch_or(ctl + kCtlStatus, bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Watchdog: latch the status bit and, for the first one, what was waited on
// (site 1 = decode dependency flag, 2 = closure entry, 3 = closure end).
__device__ __forceinline__ void watchdog(uint32_t* ctl, uint32_t site, uint32_t a, uint32_t b,
                                         uint32_t seen, uint32_t want) {
  if (__hip_atomic_fetch_or(ctl + kCtlStatus, kStWatchdog, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kStWatchdog) return;
  ctl[kCtlDiag + 0] = site;
  ctl[kCtlDiag + 1] = a;
  ctl[kCtlDiag + 2] = b;
  ctl[kCtlDiag + 3] = seen;
  ctl[kCtlDiag + 4] = want;
}

// True once any wait of the current call has timed out: every later wait
// gives up at once, so a call that cannot finish ends after one time-out.
__device__ __forceinline__ bool watchdog_fired(const uint32_t* ctl) {
  return __hip_atomic_load(const_cast<uint32_t*>(ctl) + kCtlStatus, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kStWatchdog;
}

// One stream record header (wave-uniform fields).
struct Stream {
  uint32_t mode, csym, K, n, nw, blen, body;
};

// Parse and check the record at *off (16-byte aligned) of the LDS copy `hp` of
// the first hlen payload bytes; records end within plen.  With `staged` the
// whole record must lie in the copy (the short streams are decoded from it).
// No early return and the group word counts apart (counts_ok): the four
// records' headers are a chain of LDS reads as it is.
__device__ __forceinline__ bool parse_stream(const uint8_t* hp, uint32_t hlen, uint32_t plen,
                                             uint32_t* off, uint32_t want, uint32_t maxK,
                                             bool staged, Stream& s) {
  bool ok = *off + 16 <= hlen;
  const u32x4 h = *reinterpret_cast<const u32x4*>(hp + (ok ? *off : 0u));
  const uint32_t hx = uni(h[0]);
  s.mode = hx & 0xFFu;
  s.csym = (hx >> 8) & 0xFFu;
  s.K = hx >> 16;
  s.n = uni(h[1]);
  s.nw = uni(h[2]);
  s.blen = uni(h[3]);
  s.body = *off + 16;
  const uint64_t end = (uint64_t)s.body + s.blen;
  ok = ok && s.n == want && !(staged && end > hlen);
  const uint32_t G = (s.K + 63) >> 6;
  bool fits;
  switch (s.mode) {
    case kModeEmpty: fits = !s.n && !s.blen; break;
    case kModeConst: fits = s.n && !s.blen; break;
    case kModeRaw: fits = s.blen == s.n && end <= plen; break;
    case kModeRans:
      fits = s.K >= 1 && s.K <= maxK && s.n && end <= plen &&
             (uint64_t)s.blen == 4ull * s.K + 4ull * G + 2ull * s.nw &&
             (uint64_t)s.body + 4ull * s.K + 4ull * G <= hlen;
      break;
    default: fits = false;
  }
  ok = ok && fits;
  if (ok) *off = s.body + ((s.blen + 15u) & ~15u);
  return ok;
}

// The word counts of a record's groups (at most four) add up.  The counts lie
// in the copy (parse_stream); a read of sixteen bytes from there may run past
// it, but not past the LDS it lies in.
__device__ __forceinline__ bool counts_ok(const uint8_t* hp, const Stream& s) {
  const bool rans = s.mode == kModeRans;
  const uint32_t G = (s.K + 63) >> 6;
  const u32x4 c = ld128(hp + (rans ? s.body + 4 * s.K : 0u));
  uint64_t sum = 0;
#pragma unroll
  for (uint32_t g = 0; g < kWaves; g++) sum += g < G ? c[g] : 0u;
  return !rans | (uni(sum == s.nw) != 0);
}

// The owner of slot u of a short stream (an index of sym[]), its first slot
// and its number of slots.  The bucket of u (2^bs slots) names the owner of
// its first slot; the owner of u is that or one of the next symbols that
// occur, whose first slots one read brings, so that a symbol takes two LDS
// round trips, hardly ever more.  (Over all symbols, those that never occur
// had to be stepped over one read each: 5.6 k cycles for a FASTQ block's CMD
// stream against 1.7 k for its OFF stream, twice as long.)
struct Slot {
  uint32_t k, c0, f;
};
__device__ __forceinline__ Slot bucket_sym(const uint16_t* cum, const uint8_t* bkt, uint32_t bs, uint32_t u) {
  uint32_t s = bkt[u >> bs];
  const u32x4 v = ld128(reinterpret_cast<const uint8_t*>(cum + s));     // cum[s .. s + 7]
  uint32_t c0 = v[0] & 0xFFFFu, c1 = v[0] >> 16;
#pragma unroll
  for (uint32_t k = 2; k < 8; k++) {
    const bool on = c1 <= u;              // false from the owner on: cum[256] is above every slot
    c0 = on ? c1 : c0;
    s += on ? 1u : 0u;
    c1 = on ? (k & 1 ? v[k / 2] >> 16 : v[k / 2] & 0xFFFFu) : c1;
  }
  while (c1 <= u && s < 255) {
    s++;
    c0 = c1;
    c1 = cum[s + 1];
  }
  return Slot{min(s, 255u), c0, c1 - c0};
}

// Decode a short rANS stream (one group of K <= 64 lanes) with one wave.  The
// record lies in the LDS copy `body`, so words are read from there directly.
// Lane k decodes the run of consecutive symbols starting at k*R + min(k, e),
// R = n / K, e = n mod K (container lane layout); round r decodes symbol r of
// every run still going, renormalisation words are taken in ascending lane
// order within a round.  `put.start(i)` positions lane state at symbol i and
// `put(v)` stores the lane's next symbol.  True if every state ends at 2^16 and
// every word of the group was read.
template <class Put>
__device__ bool short_rans(const uint8_t* body, const Stream& s, uint32_t P, const uint16_t* cum,
                           const uint8_t* sym, const uint8_t* bkt, uint32_t bs, Put& put) {
  const uint32_t lane = lane_id();
  const uint32_t K = s.K, n = s.n;
  const bool lane_ok = lane < K;
  const uint32_t nwg = uni(*reinterpret_cast<const uint32_t*>(body + 4 * K));
  const uint16_t* W = reinterpret_cast<const uint16_t*>(body + 4 * K + 4);
  const uint32_t lastw = nwg ? nwg - 1 : 0;
  uint32_t x = lane_ok ? *reinterpret_cast<const uint32_t*>(body + 4 * lane) : kL;
  bool ok = x >= kL && nwg == s.nw;
  const uint32_t R = n / K, e = n - R * K;
  put.start(lane * R + min(lane, e));
  const uint32_t mask = (1u << P) - 1;
  uint32_t pos = 0;
  auto round = [&](bool act) {
    if (act) {
      const uint32_t u = x & mask;
      const Slot o = bucket_sym(cum, bkt, bs, u);
      x = __umul24(o.f, x >> P) + (u - o.c0);
      put(sym[o.k]);
    }
    const bool need = act && x < kL;
    const uint64_t bal = __ballot(need);
    if (need) x = (x << 16) | (uint32_t)W[min(pos + mbcnt(bal), lastw)];
    pos += (uint32_t)__popcll(bal);
  };
  for (uint32_t r = 0; r < R; r++) round(lane_ok);
  if (e) round(lane_ok && lane < e);
  ok = ok && (!lane_ok || x == kL) && pos == nwg;
  return __ballot(!ok) == 0;
}

// The first kPreSlices 128-word slices of a literal group, its lanes' initial
// states and its word range, loaded right after the stream headers are parsed
// so that their HBM latency is spent on stages 1 and 2.  Word loads are
// clamped into the group (a group without words reads the first state
// instead), so every load stays inside the record; a corrupt stream that
// consumes more words than the group holds fails pos == nwg.
constexpr uint32_t kPreSlices = 3;
struct LitPre {
  uint32_t w[2 * kPreSlices];   // w[2 s + h] = word 128 s + 64 h + lane
  uint32_t x, woff, nwg;
};

__device__ __forceinline__ const uint16_t* lit_words(const uint8_t* body, uint32_t K, const LitPre& L) {
  const uint32_t G = (K + 63) >> 6;
  return L.nwg ? reinterpret_cast<const uint16_t*>(body + 4 * K + 4 * G) + L.woff
               : reinterpret_cast<const uint16_t*>(body);
}

// body: the record body in HBM; woff, nwg: the group's first word and word
// count (prefix sums of the group word counts, done when the block was
// prepared)
__device__ __forceinline__ void lit_prefetch(const uint8_t* body, uint32_t K, uint32_t g,
                                             uint32_t woff, uint32_t nwg, LitPre& L) {
  const uint32_t lane = lane_id(), k = (g << 6) + lane;
  L.woff = woff;
  L.nwg = nwg;
  const uint16_t* W = lit_words(body, K, L);
  const uint32_t lastw = L.nwg ? L.nwg - 1 : 0;
#pragma unroll
  for (uint32_t i = 0; i < 2 * kPreSlices; i++) L.w[i] = (uint32_t)W[min(64 * i + lane, lastw)];
  L.x = k < K ? ld32(body + 4 * k) : kL;
}

// Literal stream, one 64-lane group g of K lanes, every lane active for R
// rounds (a full group) or under `act` masks (FULL false).  Same symbols,
// words and checks as short_rans; the group's 16-bit words are staged from HBM
// through the wave's LDS ring (two 128-word slices, the next two slices in
// registers), and every staged word carries the table entry of the slot it
// starts (after x = (x << 16) | w the next slot is w mod 2^P), so a round
// makes one LDS round trip: renormalising lanes read word and entry, the
// others look up their new slot.  Each symbol goes straight to its tile
// position tp; when tp reaches the end of the lane's current literal run
// (tpend) the lane moves to the next sequence that has literals.
template <uint32_t P, bool FULL>
__device__ bool lit_group(const uint8_t* body, uint32_t K, uint32_t n, uint32_t nw_total, uint32_t g,
                          Smem& S, uint32_t wv, uint32_t ns, const LitPre& L) {
  const uint32_t lane = lane_id();
  const uint32_t k = (g << 6) + lane;
  const bool lane_ok = k < K;
  const uint32_t nwg = L.nwg;
  const uint16_t* W = lit_words(body, K, L);
  const uint32_t lastw = nwg ? nwg - 1 : 0;
  auto ldw = [&](uint32_t idx) -> uint32_t { return (uint32_t)W[min(idx, lastw)]; };
  constexpr uint32_t mask = (1u << P) - 1;
  uint16_t* ring = S.ring[wv];
  uint32_t* ringe = S.ringe[wv];
  const uint32_t* ent = S.lut;
  const uint32_t first = kLutLit + 256 * wv;           // this wave's ring, as an index of ent
  const uint16_t* words = &S.ring[0][0] - kLutLit;     // ... and of words
  uint32_t x = L.x;
  bool ok = x >= kL && L.woff + nwg <= nw_total;
  // slices 0 and 1 into the ring, slices 2..5 wait in registers
  {
    uint32_t en[4];
#pragma unroll
    for (uint32_t q = 0; q < 4; q++) en[q] = S.lut[L.w[q] & mask];
#pragma unroll
    for (uint32_t q = 0; q < 4; q++) {
      ring[64 * q + lane] = (uint16_t)L.w[q];
      ringe[64 * q + lane] = en[q];
    }
  }
  // slice 2 waits in registers (u0, u1); staging it loads the next slice
  // straight into the same registers, so no register moves follow the loads
  // and their wait falls one slice later
  static_assert(kPreSlices == 3, "the ring holds slices 0 and 1, registers slice 2");
  uint32_t u0 = L.w[4], u1 = L.w[5];
  uint32_t e = S.lut[x & mask];
  uint32_t pos = 0;
  const uint32_t R = n / K, ex = n - R * K;
  // the lane's first literal i0 lies in sequence j: lit[j] <= i0 < lit[j+1]
  const uint32_t i0 = min(k * R + min(k, ex), n ? n - 1 : 0);
  uint32_t j = 0;
  {
    uint32_t lo = 0, hi = ns - 1;
    while (lo < hi) {
      const uint32_t mid = (lo + hi + 1) >> 1;
      if (S.lit[mid] <= i0) lo = mid; else hi = mid - 1;
    }
    j = lo;
  }
  uint32_t tp = i0 - S.lit[j] + S.out[j];
  uint32_t tpend = S.out[j] + (uint32_t)S.lit[j + 1] - S.lit[j];
  // literal runs of the next three sequences in registers (start, end in the
  // tile), so that moving to the next run reads no LDS; jq = last queued one
  uint32_t q1, e1, q2, e2, q3, e3, jq = min(j + 3, ns - 1);
  {
    const uint32_t j1 = min(j + 1, ns - 1), j2 = min(j + 2, ns - 1), j3 = jq;
    q1 = S.out[j1]; e1 = q1 + (uint32_t)S.lit[j1 + 1] - S.lit[j1];
    q2 = S.out[j2]; e2 = q2 + (uint32_t)S.lit[j2 + 1] - S.lit[j2];
    q3 = S.out[j3]; e3 = q3 + (uint32_t)S.lit[j3 + 1] - S.lit[j3];
  }
  auto round = [&](bool act) {
    if (act) {
      S.tile[tp] = (uint8_t)e;
      x = __umul24((e >> 8) & 0xFFFu, x >> P) + (e >> 20);
      tp++;
    }
    const bool need = act && x < kL;
    const uint64_t bal = __ballot(need);
    const uint32_t q = (__builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32),
                                                  __builtin_amdgcn_mbcnt_lo((uint32_t)bal, pos)) & 255u) | first;
    const uint32_t w = words[q];
    // a select made of bits: of two conditions the compiler makes a branch,
    // and the two reads follow each other
    const uint32_t sel = 0u - (uint32_t)need;
    e = ent[((q ^ (x & mask)) & sel) ^ (x & mask)];
    x = need ? (x << 16) | w : x;
    pos += (uint32_t)__popcll(bal);
    // end of the lane's literal run in this sequence: the next sequence
    // with literals (every literal index below n_lit has one), from the
    // register queue while it lasts, else from the tables
    if (act && tp == tpend) {
      for (uint32_t hop = 0; hop < 3 && tp == tpend; hop++) {
        tp = q1; tpend = e1;
        q1 = q2; e1 = e2;
        q2 = q3; e2 = e3;
        q3 = e3;                          // empty run: exhausts the queue
      }
      if (tp == tpend) {
        uint32_t nj = jq + 1;
        while (nj + 1 < ns && S.lit[nj + 1] == S.lit[nj]) nj++;
        jq = min(nj, ns - 1);
        tp = S.out[jq];
        tpend = tp + (uint32_t)S.lit[jq + 1] - S.lit[jq];
        q1 = q2 = q3 = e1 = e2 = e3 = tpend;
      }
    }
  };
  // Two rounds use up at most a slice of 128 words, and two are staged: after
  // every second round, once slice s0+1 is entered, slice s0+2 goes from the
  // registers into the ring half of slice s0, and slice s0+kPreSlices is loaded
  // into them. Written out in this scope: inside the round helper, which takes
  // its state by reference, the registers would be spilled to a private array.
#define LZ_STAGE()                                                      \
    if ((pos >> 7) != s0) {                                             \
      __builtin_amdgcn_wave_barrier(); /* every lane read slice s0 */   \
      const uint32_t d = ((s0 & 1) << 7) + lane;                        \
      const uint32_t b3 = (s0 + kPreSlices) << 7;                       \
      const uint32_t ea = S.lut[u0 & mask], eb = S.lut[u1 & mask];      \
      ring[d] = (uint16_t)u0;                                           \
      ring[d + 64] = (uint16_t)u1;                                      \
      ringe[d] = ea;                                                    \
      ringe[d + 64] = eb;                                               \
      if (b3 < nwg) {                  /* words left to fetch */        \
        u0 = ldw(b3 + lane);                                            \
        u1 = ldw(b3 + 64 + lane);                                       \
      }                                                                 \
    }
  const bool on = FULL || lane_ok;
  for (uint32_t r = 0; r + 1 < R; r += 2) {
    const uint32_t s0 = pos >> 7;
    round(on);
    round(on);
    LZ_STAGE()
  }
  if (R & 1) {
    const uint32_t s0 = pos >> 7;
    round(on);
    LZ_STAGE()
  }
  if (ex) round(lane_ok && k < ex);     // no read follows: nothing to stage
#undef LZ_STAGE
  ok = ok && (!lane_ok || x == kL) && pos == nwg;
  return __ballot(!ok) == 0;
}

template <uint32_t P>
__device__ bool lit_group_p(const uint8_t* body, uint32_t K, uint32_t n, uint32_t nw, uint32_t g,
                            Smem& S, uint32_t wv, uint32_t ns, const LitPre& L) {
  if ((g << 6) + 64 <= K) return lit_group<P, true>(body, K, n, nw, g, S, wv, ns, L);
  return lit_group<P, false>(body, K, n, nw, g, S, wv, ns, L);
}

// Source byte at absolute position a (an earlier block): direct mode reads the
// whole-file output; request mode goes through the per-block address table.
__device__ __forceinline__ uint32_t src_byte(const DevArgs& A, uint64_t a, bool& bad) {
  const uint8_t* p = A.out + a;
  if (A.addr) {
    const uint64_t base = A.addr[a >> A.bl];
    if (!base) { bad = true; return 0; }
    p = reinterpret_cast<const uint8_t*>(base) + (a & ((1ull << A.bl) - 1));
  }
  return A.flow == 2 ? __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : *p;
}

// Sixteen bytes of a finished block.  With shared lines (A.flow 2) by loads
// that every XCD's writes are seen by: the aligned words that hold the bytes
// (inside the block, whose size and place are multiples of 8).
__device__ __forceinline__ u32x4 done16(const DevArgs& A, const uint8_t* p) {
  if (A.flow != 2) return ld128(p);
  const uint32_t o = (uint32_t)(uintptr_t)p & 7u;
  const uint64_t* q = reinterpret_cast<const uint64_t*>(p - o);
  uint64_t w[3];
#pragma unroll
  for (uint32_t k = 0; k < 3; k++)
    w[k] = k < 2 || o ? __hip_atomic_load(q + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
  const uint64_t lo = o ? (w[0] >> (8 * o)) | (w[1] << (64 - 8 * o)) : w[0];
  const uint64_t hi = o ? (w[1] >> (8 * o)) | (w[2] << (64 - 8 * o)) : w[1];
  return u32x4{(uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32)};
}

// Sixteen source bytes from position a (all in earlier blocks).  In request
// mode two blocks at most, whose decoded bytes may lie anywhere: bytes on both
// sides of the block edge are fetched one by one.
__device__ __forceinline__ u32x4 src16(const DevArgs& A, uint64_t a, bool& bad) {
  if (!A.addr) return done16(A, A.out + a);
  const uint64_t base = A.addr[a >> A.bl], in = a & ((1ull << A.bl) - 1);
  if (!base) {
    bad = true;
    return u32x4{};
  }
  if (in + 16 <= (1ull << A.bl)) return done16(A, reinterpret_cast<const uint8_t*>(base) + in);
  u32x4 v = {};
#pragma unroll 1
  for (uint32_t k = 0; k < 16; k++) {
    const uint32_t x = src_byte(A, a + k, bad) << (8 * (k & 3));
#pragma unroll
    for (uint32_t w = 0; w < 4; w++) v[w] |= w == (k >> 2) ? x : 0u;
  }
  return v;
}

// Inclusive scan over the 64 lanes of a wave with DPP moves (no LDS): shifts
// by 1, 2, 4 and 8 inside each 16-lane row, then the last lane of row 0 is
// added to row 1 and of row 2 to row 3 (row_bcast:15), then lane 31 to rows
// 2 and 3 (row_bcast:31).  Lanes whose DPP source is outside the row read 0.
__device__ __forceinline__ uint32_t wave_scan(uint32_t v) {
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);   // row_shr:1
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);   // row_shr:2
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);   // row_shr:4
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);   // row_shr:8
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);   // row_bcast:15
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);   // row_bcast:31
  return v;
}

// Block-wide exclusive scans of three counts at once; tot[] receives the sums.
__device__ void block_scan3(Smem& S, const uint32_t v[3], uint32_t pre[3], uint32_t tot[3]) {
  const uint32_t lane = lane_id(), wv = threadIdx.x >> 6;
  uint32_t incl[3];
#pragma unroll
  for (int f = 0; f < 3; f++) {
    incl[f] = wave_scan(v[f]);
    if (lane == 63) S.scan[f][wv] = incl[f];
  }
  __syncthreads();
#pragma unroll
  for (int f = 0; f < 3; f++) {
    uint32_t base = 0, all = 0;
#pragma unroll
    for (uint32_t q = 0; q < kWaves; q++) {
      const uint32_t w = S.scan[f][q];
      if (q < wv) base += w;
      all += w;
    }
    pre[f] = base + incl[f] - v[f];
    tot[f] = all;
  }
  // no closing barrier: S.scan is next written by the next block's scan,
  // many barriers later
}

// Small-stream symbol lookup: binary search of slot u in a 257-entry
// cumulative table.
__device__ __forceinline__ uint32_t search_sym(const uint16_t* cum, uint32_t u) {
  uint32_t lo = 0;
#pragma unroll
  for (uint32_t step = 128; step; step >>= 1)
    if (cum[lo + step] <= u) lo += step;
  return lo;
}

// Writes the decoded values of a short stream: symbol i is byte plane i / ns
// of value i mod ns (values stored byte-plane major); a lane's symbols are
// consecutive, so its (plane, index) pair advances by one each call.
struct PutPlanes {
  uint8_t* lo;      // planes 0..lo_planes-1: byte `plane` of the value at lo + stride * idx
  uint8_t* hi;      // plane 4 (offsets only): hi[idx]
  uint32_t stride, ns, idx, plane;
  __device__ void start(uint32_t i) {
    plane = i / ns;
    idx = i - plane * ns;
  }
  __device__ void operator()(uint32_t v) {
    if (plane < 4) lo[stride * idx + min(plane, stride - 1)] = (uint8_t)v;
    else hi[idx] = (uint8_t)v;
    if (++idx == ns) { idx = 0; plane++; }
  }
};

// Where block b's payload lies and how many sequences and literals it holds.
struct BlockDir {
  uint64_t poff;
  uint32_t plen, ns, nlit, blen;
};

__device__ __forceinline__ BlockDir block_dir(const DevArgs& A, uint32_t b) {
  const uint64_t B = 1ull << A.bl, sb = (uint64_t)b << A.bl;
  const uint8_t* de = A.arc + A.off_dir + (uint64_t)b * kDirEntry;
  BlockDir d;
  d.poff = ld64(de);
  d.plen = ld32(de + 8);
  d.ns = ld32(de + 12);
  d.nlit = ld32(de + 16);
  d.blen = (uint32_t)((sb + B <= A.n) ? B : A.n - sb);
  return d;
}

// The first n of the four stream records (CMD, MLEN, OFF, LIT) parsed and
// checked from the LDS copy hp of the block's first hlen payload bytes (every
// thread parses the same bytes, so the result is wave-uniform).
__device__ __forceinline__ bool parse_records(const DevArgs& A, const BlockDir& d, const uint8_t* hp,
                                              uint32_t hlen, uint32_t n, Stream& sc, Stream& sm,
                                              Stream& so, Stream& sl) {
  uint32_t off = 0;
  bool ok = d.ns >= 1 && d.ns <= kMaxSeq && d.nlit <= d.blen && (d.poff & 15) == 0;
  ok &= parse_stream(hp, hlen, d.plen, &off, 2 * d.ns, A.seq_lanes, true, sc);
  if (n > 1) ok &= parse_stream(hp, hlen, d.plen, &off, 2 * d.ns, A.seq_lanes, true, sm);
  if (n > 2) {
    ok &= parse_stream(hp, hlen, d.plen, &off, A.w * d.ns, A.seq_lanes, true, so);
    ok &= parse_stream(hp, hlen, d.plen, &off, d.nlit, A.lit_lanes, false, sl);
  }
  if (!ok) return false;
  ok = counts_ok(hp, sc);
  if (n > 1) ok &= counts_ok(hp, sm);
  if (n > 2) {
    const bool a = counts_ok(hp, so), b = counts_ok(hp, sl);
    ok &= a & b;
  }
  return ok;
}

// Short stream `role` of a block with ns sequences, by one wave: 0 CMD ->
// lit[] (LL), 1 MLEN -> out[] (ML), 2 OFF -> oflo/ofhi (absolute offsets).
__device__ bool short_stream(Smem& S, const DevArgs& A, uint32_t role, const Stream& s,
                             const uint8_t* hp, uint32_t ns) {
  const uint32_t lane = lane_id();
  PutPlanes put;
  put.ns = ns;
  if (role < 2) {
    put.lo = role == 0 ? reinterpret_cast<uint8_t*>(S.lit) : reinterpret_cast<uint8_t*>(S.out);
    put.hi = put.lo;
    put.stride = 2;
  } else {
    put.lo = reinterpret_cast<uint8_t*>(S.oflo);
    put.hi = S.ofhi;
    put.stride = 4;
    // offsets narrower than 5 bytes: clear the planes the stream does not hold
    for (uint32_t j = lane; j < ns; j += 64) { S.oflo[j] = 0; S.ofhi[j] = 0; }
    __builtin_amdgcn_wave_barrier();
  }
  if (s.mode == kModeRans) {
    const uint32_t P = A.P[1 + role];                 // at least 8
    return short_rans(hp + s.body, s, P, S.cum[role], S.sym[role], S.bkt[role], P - 7, put);
  }
  if (s.mode == kModeRaw || s.mode == kModeConst) {
    const uint8_t* src = hp + s.body;
    for (uint32_t i = lane; i < s.n; i += 64) {
      put.start(i);
      put(s.mode == kModeRaw ? (uint32_t)src[i] : s.csym);
    }
  }
  return true;
}

// What the later stages need of the prepared block (one thread): its
// directory fields, the literal record and the literal groups' word ranges
// (the group word counts lie in the copy hp: parse_stream checks that).
__device__ __forceinline__ void put_prep(Smem& S, const BlockDir& d, const Stream& s, const uint8_t* hp,
                                         bool ok) {
  S.pdir[0] = (uint32_t)d.poff; S.pdir[1] = (uint32_t)(d.poff >> 32); S.pdir[2] = d.ns; S.pdir[3] = d.nlit;
  S.pst[0] = s.mode; S.pst[1] = s.csym; S.pst[2] = s.K; S.pst[3] = s.n;
  S.pst[4] = s.nw; S.pst[5] = s.blen; S.pst[6] = s.body;
  const uint32_t G = ok && s.mode == kModeRans ? (s.K + 63) >> 6 : 0u;
  const uint32_t* cnt = reinterpret_cast<const uint32_t*>(hp + s.body + 4 * s.K);
  uint32_t w = 0;
  for (uint32_t g = 0; g < kWaves; g++) {
    const uint32_t c = g < G ? cnt[g] : 0u;
    S.plw[g] = w;
    S.pln[g] = c;
    w += c;
  }
}

__device__ __forceinline__ uint32_t take_ticket(const DevArgs& A) {
  return __hip_atomic_fetch_add(A.ctl + kCtlTicket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Stages 0 and 1 of block b ("preparing" it): the payload prefix is copied
// into LDS, the four stream records are parsed and checked, and the CMD, MLEN
// and OFF streams are decoded into the sequence tables.  The literal record
// goes to S.pst with the directory fields and literal group word ranges
// (put_prep), the outcome to S.pok; a short stream that fails its checks sets
// S.perr[k] (written by the wave that decoded stream k, 0 or 1).
//
// How many blocks b copies from, where their list starts, and whether any
// block copies from b.  Only by-ticket launches need them.
struct Deps {
  uint64_t at;
  uint32_t n, used;
};
__device__ __forceinline__ Deps block_deps(const DevArgs& A, uint32_t b) {
  Deps d = {0, 0, 0};
  if (A.flow) {
    d.used = A.flags[b] != kFlagLeaf ? 1u : 0u;
    d.at = ld64(A.arc + A.off_dep_ptr + 8ull * b);
    d.n = (uint32_t)(ld64(A.arc + A.off_dep_ptr + 8ull * b + 8) - d.at);
  }
  return d;
}
__device__ __forceinline__ uint32_t dep_id(const DevArgs& A, const Deps& d, uint32_t i) {
  return ld32(A.arc + A.off_dep_idx + 4 * (d.at + i));
}
// by one wave
__device__ __forceinline__ void put_deps(Smem& S, const DevArgs& A, const Deps& d) {
  const uint32_t lane = lane_id();
  for (uint32_t i = lane; i < min(d.n, kDeps); i += 64) S.dep[i] = dep_id(A, d, i);
  if (lane == 0) {
    S.ndep = d.n;
    S.used = d.used;
    S.wait = 0;
  }
}

// prep_tile: all four waves.  The first min(plen, 16 KiB) payload bytes go
// into the tile (free until the literal stage) with one round of 16-byte
// loads; waves 0..2 decode the short streams from there (at most about 9.3 KB
// with their headers for 1025 sequences).  Corrupt records are latched.
__device__ __forceinline__ void prep_tile(Smem& S, const DevArgs& A, uint32_t b) {
  const uint32_t t = threadIdx.x, wv = uni(t >> 6), lane = lane_id();
  const BlockDir d = block_dir(A, b);
  const Deps dp = block_deps(A, b);
  const uint8_t* pay = A.arc + A.off_payload + d.poff;
  CLK_START(S);
  const uint32_t hlen = min(d.plen, kB);
  {
    const uint32_t n16 = hlen >> 4;
    const bool tail = t < (hlen & 15u);              // bytes past the last 16
    const uint32_t tb = tail ? (uint32_t)pay[(hlen & ~15u) + t] : 0u;
    if (((uintptr_t)pay & 15u) == 0) {   // straight into LDS, one HBM round trip
#pragma unroll 1
      for (uint32_t i = 0; i < kB / (16 * kWG); i++)
        if (t + kWG * i < n16) lds_dma16(pay + 16 * (t + kWG * i), S.tile + 16 * (64 * wv + kWG * i));
      vm_wait();
    } else {
      const uint4* src4 = reinterpret_cast<const uint4*>(pay);
      uint4* dst4 = reinterpret_cast<uint4*>(S.tile);
      for (uint32_t c = t; c < n16; c += kWG) dst4[c] = src4[c];
    }
    if (tail) S.tile[(hlen & ~15u) + t] = (uint8_t)tb;
  }
  if (t == 0) S.next = 0;
  if (wv == 3) put_deps(S, A, dp);
  __syncthreads();
  CLK_MARK(S, 0);
  Stream sc, sm, so, sl;
  const bool ok = parse_records(A, d, S.tile, hlen, 4, sc, sm, so, sl);
  if (t == 0) {
    S.pok = ok ? 1u : 0u;
    put_prep(S, d, sl, S.tile, ok);
    if (!ok) latch(A.ctl, kStCorrupt);
  }
  CLK_MARK(S, 1);
  if (ok && wv < 3) {
    const Stream& s = wv == 0 ? sc : (wv == 1 ? sm : so);
    const bool okw = short_stream(S, A, wv, s, S.tile, d.ns);
    if (lane == 0) S.perr[wv] = okw ? 0u : 1u;
  }
  __syncthreads();
  CLK_MARK(S, 2);
}

// prep_ring: waves 1..3 only, while wave 0 resolves the previous block's
// in-block matches, so no workgroup barrier may be used.  Every wave copies
// the same first kPrepRing payload bytes into the literal rings (idle from
// the end of the literal stage to the next one) itself, so each needs only
// its own stores before it reads; waves 1..3 decode CMD, MLEN and OFF.  A
// prefix too short for the short streams and the literal record's states and
// counts (or corrupt records) leaves S.pok 0, and the block is prepared again
// by prep_tile.  The caller guarantees that the sequence tables, S.pst and
// the rings are not in use.
__device__ __forceinline__ void prep_ring(Smem& S, const DevArgs& A, uint32_t b) {
  const uint32_t wv = uni(threadIdx.x >> 6), lane = lane_id();
  const BlockDir d = block_dir(A, b);
  const Deps dp = block_deps(A, b);
  const uint8_t* pay = A.arc + A.off_payload + d.poff;
  const uint32_t hlen = min(d.plen, kPrepRing);
  {
    const uint32_t n16 = hlen >> 4;
    const bool tail = lane < (hlen & 15u);           // bytes past the last 16
    const uint32_t tb = tail ? (uint32_t)pay[(hlen & ~15u) + lane] : 0u;
    if (((uintptr_t)pay & 15u) == 0) {
      // every 1 KiB of the prefix at once, straight into LDS: one HBM round
      // trip (copied through registers it was one per 1 KiB, as the
      // registers are all taken here)
#pragma unroll 1
      for (uint32_t i = 0; i < kPrepRing / 1024; i++)   // not unrolled: no hoisted addresses
        if (lane + 64 * i < n16) lds_dma16(pay + 16 * (lane + 64 * i), S.prep + 1024 * i);
    } else {
      const uint4* src4 = reinterpret_cast<const uint4*>(pay);
      uint4* dst4 = reinterpret_cast<uint4*>(S.prep);
      for (uint32_t c = lane; c < n16; c += 64) dst4[c] = src4[c];
    }
    if (wv == 3) put_deps(S, A, dp);
    vm_wait();
    if (tail) S.prep[(hlen & ~15u) + lane] = (uint8_t)tb;
  }
  __builtin_amdgcn_wave_barrier();
  Stream sc, sm, so, sl;
  // each wave as many records as it needs; wave 3, whose OFF stream is mostly
  // stored and soon done, all four and the bookkeeping
  const uint32_t role = wv - 1;
  const bool ok = parse_records(A, d, S.prep, hlen, role < 2 ? role + 1 : 4u, sc, sm, so, sl);
  bool okw = true;
  if (ok) {
    const Stream& s = role == 0 ? sc : (role == 1 ? sm : so);
    okw = short_stream(S, A, role, s, S.prep, d.ns);
  }
  if (ok && lane == 0) S.perr[role] = okw ? 0u : 1u;
  if (wv == 3 && lane == 0) {
    S.pok = ok ? 1u : 0u;
    put_prep(S, d, sl, S.prep, ok);
    S.next = 0;
  }
}

// n bytes of the tile from src to dst by one wave, not overlapping: 16 bytes a
// lane at any alignment, 2 KiB of loads before their stores.
__device__ __forceinline__ void tile_copy(Smem& S, uint32_t dst, uint32_t src, uint32_t n) {
  const uint32_t o = 16 * lane_id();
  for (uint32_t c = 0; c < n; c += 2048) {
    u32x4 v[2] = {};
#pragma unroll
    for (uint32_t u = 0; u < 2; u++)
      if (c + 1024 * u + o < n) v[u] = ld128(S.tile + src + c + 1024 * u + o);
#pragma unroll
    for (uint32_t u = 0; u < 2; u++) {
      const uint32_t k = c + 1024 * u + o;
      if (k < n) st_upto16(S.tile + dst + k, v[u], min(16u, n - k));
    }
  }
}

// In-block match of M bytes to tile position d0 from s = d0 - d (s < 0: its
// first bytes lie in earlier blocks), by one wave: the d (or M) bytes before
// the match repeats itself are copied, then what is there is appended to
// itself, doubling, until M bytes stand; a period that divides 16 is laid out
// in a register and stored.  A match that fills its block with period 2 was
// 27 us of a block's 55 byte by byte, 64 at a time and each step waiting for
// the one before.
__device__ __forceinline__ void copy_long(Smem& S, const DevArgs& A, uint64_t sb, uint32_t d0, uint32_t M,
                                          int32_t s, uint32_t d, bool& bad) {
  const uint32_t lane = lane_id();
  const uint32_t n = min(d, M), n0 = s < 0 ? min(n, (uint32_t)-s) : 0u;
  for (uint32_t c = 0; c < n0; c += 512) {          // from earlier blocks, eight loads in flight
    uint32_t v[8];
#pragma unroll
    for (uint32_t u = 0; u < 8; u++) {
      const uint32_t k = c + 64 * u + lane;
      v[u] = k < n0 ? src_byte(A, sb + (int64_t)s + k, bad) : 0u;
    }
#pragma unroll
    for (uint32_t u = 0; u < 8; u++) {
      const uint32_t k = c + 64 * u + lane;
      if (k < n0) S.tile[d0 + k] = (uint8_t)v[u];
    }
  }
  if (n > n0) tile_copy(S, d0 + n0, (uint32_t)(s + (int32_t)n0), n - n0);
  if (d < M && d <= 16 && (d & (d - 1)) == 0) {
    // a period that divides 16: every 16 bytes are the same
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const u32x4 w = ld128(S.tile + d0);
    const uint32_t x = d == 1 ? (w[0] & 0xFFu) * 0x01010101u : (d == 2 ? (w[0] & 0xFFFFu) * 0x00010001u : w[0]);
    const uint32_t y = d >= 8 ? w[1] : x;
    const u32x4 v = {x, y, d == 16 ? w[2] : x, d == 16 ? w[3] : y};
    for (uint32_t k = 16 * lane; k < M; k += 1024) st_upto16(S.tile + d0 + k, v, min(16u, M - k));
    return;
  }
  for (uint32_t f = n; f < M; f += min(f, M - f)) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // reads what was written
    tile_copy(S, d0 + f, d0, min(f, M - f));
  }
}

// Decode block b, prepared by prep_tile or prep_ring (S.pok, S.pst and the
// sequence tables hold its stages 0 and 1), into the LDS tile and store it.
// it: its place in the queue's `total` blocks from qb on; epoch: the value of
// a finished block's flag.  The next place and block go to S.nit and S.nb
// (kNext of the result; unset after corrupt data); kPrepared: that block has
// been prepared meanwhile, by waves 1..3 while wave 0 resolved b's in-block
// matches; kUsed: this block is still to be published, if others copy from it,
// corrupt or not.  Every loop below is bounded by values read from global
// memory (directory, stream headers) or by the spin limit.
constexpr uint32_t kPrepared = 1, kNext = 2, kUsed = 4;
__device__ __forceinline__ uint32_t decode_block(Smem& S, const DevArgs& A, uint32_t b, uint32_t qb,
                                                 uint32_t total, uint32_t it, uint32_t epoch) {
  const uint32_t t = threadIdx.x, wv = uni(t >> 6), lane = lane_id();
  const uint64_t B = 1ull << A.bl, sb = (uint64_t)b << A.bl;
  const uint32_t blen = (uint32_t)((sb + B <= A.n) ? B : A.n - sb);
  if (!uni(S.pok)) return kUsed;               // corrupt records (latched by prep_tile)
  uint8_t* dst = A.addr ? reinterpret_cast<uint8_t*>(A.addr[b]) : A.out + sb;
  // completion flags of the blocks b copies from, one per thread; looked at
  // at the end of stage 2
  const uint32_t nd = A.flow ? uni(S.ndep) : 0u;
  const uint32_t dep = t < min(nd, kDeps) ? S.dep[t] : 0u;
  const bool used = A.flow && uni(S.used);
  uint32_t flag = epoch;
  if (t < min(nd, kDeps)) flag = __hip_atomic_load(A.flags + dep, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const uint64_t poff = (uint64_t)uni(S.pdir[0]) | ((uint64_t)uni(S.pdir[1]) << 32);
  const uint32_t ns = uni(S.pdir[2]), nlit = uni(S.pdir[3]);
  const uint8_t* pay = A.arc + A.off_payload + poff;
  Stream sl;
  sl.mode = uni(S.pst[0]); sl.csym = uni(S.pst[1]); sl.K = uni(S.pst[2]); sl.n = uni(S.pst[3]);
  sl.nw = uni(S.pst[4]); sl.blen = uni(S.pst[5]); sl.body = uni(S.pst[6]);
  // literal group of this wave (K <= 256: at most one per wave), fetched ahead
  const uint32_t Glit = sl.mode == kModeRans ? (sl.K + 63) >> 6 : 0u;
  LitPre lp;
  if (wv < Glit) lit_prefetch(pay + sl.body, sl.K, wv, uni(S.plw[wv]), uni(S.pln[wv]), lp);
  if (t == 0) S.err = 0;

  // ---- stage 2: command placement.  One block scan of (LL, LL + ML,
  // in-block match) counts gives literal and output positions and the order
  // of the in-block matches; the block's sequence invariants are checked.
  // Values are u16 and ns <= 1025, so no sum reaches 2^32.  A block of at
  // most 64 sequences is placed by wave 0 alone with one wave scan (no
  // workgroup barrier); waves 1..3 wait at the stage's closing barrier.
  const bool one = ns <= 64;
  if (!one || wv == 0) {
    const uint32_t per = (ns + kWG - 1) / kWG;   // <= 5
    const uint32_t j0 = min(ns, t * per), j1 = min(ns, j0 + per);
    uint32_t v[3] = {0, 0, 0};
    bool bad = false;
    // one sequence per thread up to 256 of them (loops not unrolled: for their
    // most of five iterations a thread, all the others paid)
#pragma unroll 1
    for (uint32_t j = j0; j < j1; j++) {
      const uint32_t ll = S.lit[j], ml = S.out[j];
      const uint64_t of = (uint64_t)S.oflo[j] | ((uint64_t)S.ofhi[j] << 32);
      v[0] += ll;
      v[1] += ll + ml;
      v[2] += ml && of + ml > sb ? 1u : 0u;
    }
    uint32_t pre[3], tot[3];
    if (one) {
#pragma unroll
      for (int f = 0; f < 3; f++) {
        const uint32_t incl = wave_scan(v[f]);
        pre[f] = incl - v[f];
        tot[f] = __builtin_amdgcn_readlane(incl, 63);
      }
    } else {
      block_scan3(S, v, pre, tot);
    }
    const uint32_t tl = tot[0], to = tot[1];
    bad |= tl != nlit || to != blen;
    uint32_t pl = pre[0], po = pre[1];
    uint32_t pin = pre[2];
#pragma unroll 1
    for (uint32_t j = j0; j < j1; j++) {
      const uint32_t ll = S.lit[j], ml = S.out[j];
      const uint64_t of = (uint64_t)S.oflo[j] | ((uint64_t)S.ofhi[j] << 32);
      S.lit[j] = (uint16_t)pl;
      S.out[j] = (uint16_t)po;
      if (ml == 0) {
        bad |= (j != ns - 1) || of != 0;
      } else {
        bad |= ml < A.m || of >= sb + po + ll;
        if (of + ml <= sb) {
          S.lst[atomicAdd(&S.next, 1u)] = (uint16_t)j;   // from earlier blocks, any order
        } else {
          S.lst[kMaxSeq - 1 - pin] = (uint16_t)j;        // in-block, in sequence order
          if (pin < 64) {                                // the common case: its fields at once
            const uint32_t d0 = po + ll;
            const uint64_t dabs = sb + d0;
            S.fdst[pin] = (uint16_t)d0;
            S.flen[pin] = (uint16_t)min(ml, blen);
            S.fpk[pin] = ((uint32_t)((int64_t)of - (int64_t)sb + 16384) & 0xFFFFu) |
                         ((dabs > of ? (uint32_t)min<uint64_t>(dabs - of, 32767) : 1u) << 16);
          }
          pin++;
        }
      }
      pl += ll;
      po += ll + ml;
    }
    if (t == 0) {
      S.lit[ns] = (uint16_t)min(tl, 65535u);
      S.out[ns] = (uint16_t)min(to, 65535u);
      S.nin = tot[2];
    }
    if (bad) S.err = 1;
  }
  if (64 * wv < nd) {          // this wave holds some of the flags
    if (__ballot(flag != epoch) || nd > kDeps) S.wait = 1;
  }
  __syncthreads();
  if (S.err || S.perr[0] || S.perr[1] || S.perr[2]) {
    if (t == 0) latch(A.ctl, kStCorrupt);
    return kUsed;
  }
  const bool wait = uni(S.wait) != 0;
  CLK_MARK(S, 3);

  // With at most 64 in-block matches: the earlier ones [nlo, nhi) that lane a's
  // match copies from (wave 0; stage 4a), worked out while a block waits for
  // others, or else in stage 4.
  const uint32_t cnt = min(S.nin, ns);
  uint32_t nlo = 0, nhi = 0;
  auto near_ranges = [&]() {
    // the matches that end at or before the window's start, and those that
    // start before its end: both arrays ascend, so eight of the 64 entries
    // name the group of eight that the bound lies in
    const bool have = lane < cnt;
    const uint32_t a = have ? lane : 0u, pk = S.fpk[a], dst = S.fdst[a], len = S.flen[a], d = (pk >> 16) & 0x7FFFu;
    const int32_t s = (int32_t)(pk & 0xFFFFu) - 16384, we = s + (int32_t)min(d, len);
    const uint32_t beg = have ? dst : 0xFFFFu, end = have ? dst + len : 0xFFFFu;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    S.fdst[lane] = (uint16_t)beg;
    S.frng[lane] = (uint16_t)end;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    auto below = [&](uint32_t mine, const uint16_t* all, uint32_t x) {    // entries below x
      uint32_t g = 0;
#pragma unroll
      for (uint32_t k = 0; k < 8; k++) g += __builtin_amdgcn_readlane(mine, 8 * k + 7) < x ? 1u : 0u;
      const u32x4 v = ld128(reinterpret_cast<const uint8_t*>(all + 8 * min(g, 7u)));
      uint32_t n = 8 * min(g, 7u);
#pragma unroll
      for (uint32_t k = 0; k < 4; k++) n += ((v[k] & 0xFFFFu) < x ? 1u : 0u) + ((v[k] >> 16) < x ? 1u : 0u);
      return n;
    };
    nlo = min(below(end, S.frng, (uint32_t)max(s, 0) + 1), 63u);
    nhi = min(below(beg, S.fdst, (uint32_t)max(we, 0)), 63u);
  };

  // ---- stage 3: literals straight to their tile positions; external matches
  {
    bool bad = false;
    // Matches with a source wholly in earlier blocks, four lanes a match, 16
    // bytes a lane at any alignment.  Of a match of 16 bytes or more the last
    // piece is moved back to end with the match (its overlap is written twice
    // with the same bytes), so every access is whole and inside the source.
    // The first 128 bytes of the first 64 matches are loaded before the literal
    // decode and stored after it, so that their latency is spent decoding.
    const uint32_t nx = min(S.next, ns), slot = t >> 2, sub = 16 * (t & 3);
    struct Ext {
      u32x4 v, w;           // bytes sub .. and 64 + sub ..
      uint32_t M, d0;       // match length, destination
      uint64_t of;          // source
    };
    auto ext_fields = [&](uint32_t e, Ext& x) {
      const uint32_t q = e < nx ? min((uint32_t)S.lst[e], ns - 1) : 0u;
      const uint32_t L = (uint32_t)S.lit[q + 1] - S.lit[q];
      x.M = e < nx ? (uint32_t)S.out[q + 1] - S.out[q] - L : 0u;
      x.d0 = S.out[q] + L;
      x.of = (uint64_t)S.oflo[q] | ((uint64_t)S.ofhi[q] << 32);
    };
    auto ext_load = [&](Ext& x) {
      if (x.M >= 16 && sub < x.M) x.v = src16(A, x.of + min(sub, x.M - 16), bad);
      if (64 + sub < x.M) x.w = src16(A, x.of + min(64 + sub, x.M - 16), bad);
    };
    auto ext_store = [&](const Ext& x) {
      if (x.M >= 16 && sub < x.M) st_any<u32x4>(S.tile + x.d0 + min(sub, x.M - 16), x.v);
      if (64 + sub < x.M) st_any<u32x4>(S.tile + x.d0 + min(64 + sub, x.M - 16), x.w);
    };
    Ext first;
    first.v = first.w = u32x4{};
    ext_fields(slot, first);
    if (!wait) ext_load(first);
    // the workgroup's next place; the literal decode hides the ticket's round
    // trip (several microseconds while every workgroup takes them; taken
    // during the preparation, one block further ahead, it held that up)
    uint32_t nit = it + A.nwg, nbq = ~0u;
    if (A.flow && t == 64) nit = take_ticket(A);
    if (wv < Glit) {
      const uint32_t g = wv;
      bool okg;
      switch (A.P[kLit]) {
        case 8: okg = lit_group_p<8>(pay + sl.body, sl.K, sl.n, sl.nw, g, S, wv, ns, lp); break;
        case 9: okg = lit_group_p<9>(pay + sl.body, sl.K, sl.n, sl.nw, g, S, wv, ns, lp); break;
        case 10: okg = lit_group_p<10>(pay + sl.body, sl.K, sl.n, sl.nw, g, S, wv, ns, lp); break;
        case 11: okg = lit_group_p<11>(pay + sl.body, sl.K, sl.n, sl.nw, g, S, wv, ns, lp); break;
        default: okg = lit_group_p<12>(pay + sl.body, sl.K, sl.n, sl.nw, g, S, wv, ns, lp); break;
      }
      if (!okg) bad = true;
    } else if (sl.mode == kModeRaw || sl.mode == kModeConst) {
      const uint8_t* src = pay + sl.body;
      uint32_t from = 0;
      if (sl.mode == kModeRaw && ns == 1 && ((uintptr_t)src & 15u) == 0) {
        // A stored block of one literal run: its whole 16 bytes straight into
        // the tile, all in flight at once.  (Byte by byte each thread waited
        // for one load after the other: 32 MiB of noise 67 us, so 27.)
        const uint32_t n16 = min(sl.n, kB) >> 4;
#pragma unroll 1
        for (uint32_t i = 0; i < kB / (16 * kWG); i++)
          if (t + kWG * i < n16) lds_dma16(src + 16 * (t + kWG * i), S.tile + 16 * (64 * wv + kWG * i));
        vm_wait();
        from = 16 * n16;
      }
      // one thread per literal: the sequence by binary search
      for (uint32_t i = from + t; i < sl.n; i += kWG) {
        uint32_t lo = 0, hi = ns - 1;
        while (lo < hi) {
          const uint32_t mid = (lo + hi + 1) >> 1;
          if (S.lit[mid] <= i) lo = mid; else hi = mid - 1;
        }
        const uint32_t p = i - S.lit[lo] + S.out[lo];
        S.tile[min(p, kB - 1)] = sl.mode == kModeRaw ? src[i] : (uint8_t)sl.csym;
      }
    }
    CLK_MARK(S, 4);
    if (t == 64 && nit < total) nbq = A.queue[qb + nit];
    if (wait) {
      if (wv == 0 && cnt && cnt <= 64) near_ranges();
      // The blocks b copies from have smaller tickets, so their workgroups
      // run or have finished, and none of them waits for this one.
      if (64 * wv < nd) {
        const Deps dl = block_deps(A, b);
        for (uint32_t i = t; __ballot(i < nd); i += kWG) {
          const uint32_t id = i < kDeps ? dep : (i < nd ? dep_id(A, dl, i) : 0u);
          bool pend = i < nd;
          for (uint32_t spins = 0;; spins++) {
            if (pend && __hip_atomic_load(A.flags + id, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == epoch) pend = false;
            if (!__ballot(pend)) break;
            if (spins >= A.spin_limit || ((spins & 255u) == 255u && uni(watchdog_fired(A.ctl)))) {
              if (pend) watchdog(A.ctl, 1, b, id, epoch - 1, epoch);
              break;
            }
            __builtin_amdgcn_s_sleep(1);
          }
        }
      }
      __syncthreads();
      ext_load(first);
    }
    ext_store(first);
    // what is left of a match: the bytes past 128, by its four lanes up to 1 KiB
    // and by the whole wave beyond, or a match of less than 16 bytes, byte by byte
    auto ext_rest = [&](const Ext& x) {
      if (!__ballot(x.M > 128 || x.M - 1u < 15u)) return;
      const uint32_t mid = x.M <= 1024 ? x.M : 0u;
      for (uint32_t k0 = 128 + sub; __ballot(k0 < mid); k0 += 256) {
        u32x4 v[4] = {};
#pragma unroll
        for (uint32_t u = 0; u < 4; u++)
          if (k0 + 64 * u < mid) v[u] = src16(A, x.of + min(k0 + 64 * u, mid - 16), bad);
#pragma unroll
        for (uint32_t u = 0; u < 4; u++)
          if (k0 + 64 * u < mid) st_any<u32x4>(S.tile + x.d0 + min(k0 + 64 * u, mid - 16), v[u]);
      }
      for (uint64_t big = __ballot(x.M > 1024 && sub == 0); big; big &= big - 1) {     // wave-uniform
        const uint32_t l = (uint32_t)__builtin_ctzll(big);
        const uint32_t M = __builtin_amdgcn_readlane(x.M, l), d0 = __builtin_amdgcn_readlane(x.d0, l);
        const uint64_t of = (uint64_t)__builtin_amdgcn_readlane((uint32_t)x.of, l) |
                            ((uint64_t)__builtin_amdgcn_readlane((uint32_t)(x.of >> 32), l) << 32);
        for (uint32_t c = 128 + 16 * lane; __ballot(c < M); c += 4096) {
          u32x4 v[4] = {};
#pragma unroll
          for (uint32_t u = 0; u < 4; u++)
            if (c + 1024 * u < M) v[u] = src16(A, of + min(c + 1024 * u, M - 16), bad);
#pragma unroll
          for (uint32_t u = 0; u < 4; u++)
            if (c + 1024 * u < M) st_any<u32x4>(S.tile + d0 + min(c + 1024 * u, M - 16), v[u]);
        }
      }
      const uint32_t few = x.M < 16 ? x.M : 0u;
      for (uint32_t k = t & 3; __ballot(k < few); k += 4)
        if (k < few) S.tile[x.d0 + k] = (uint8_t)src_byte(A, x.of + k, bad);
    };
    ext_rest(first);
    for (uint32_t e = 64 + slot; __ballot(e < nx); e += 64) {
      ext_fields(e, first);
      ext_load(first);
      ext_store(first);
      ext_rest(first);
    }
    if (bad) S.err = 1;
    if (t == 64) {
      S.nit = nit;
      S.nb = nbq;
    }
  }
  __syncthreads();
  if (S.err) {
    if (t == 0) latch(A.ctl, kStCorrupt);
    return kNext | kUsed;
  }
  const uint32_t nb = uni(S.nb);
  CLK_MARK(S, 5);

  // ---- stage 4: matches whose source touches the block itself.
  // With period d = p - OF, out[p+k] = out[OF + (k mod d)] for every k (the
  // byte-sequential overlap rule unrolled); only the window OF..OF+min(d,M)-1
  // is read and it is final once every earlier match writing into it is done.
  // 4a: per match a (sequence order): destination, length, block-relative
  //     source and period, and the index range of earlier in-block matches
  //     whose destinations its window meets;
  // 4b: wave 0 copies them in passes over 64-entry chunks (every earlier
  //     chunk complete): a pass takes every pending match whose predecessors
  //     are done.  Matches of at most 256 bytes with their source inside the
  //     tile that do not overlap themselves or repeat one byte are copied
  //     together, in 16-byte pieces; the others by the whole wave, one at a
  //     time.
  // With at most 64 in-block matches (the common case) stage 2 has written
  // their fields to their own small arrays and only wave 0 works on them: the
  // sequence tables are free, and waves 1..3 prepare the next block
  // meanwhile.  With more, the fields are packed into the sequence tables and
  // 4a uses every thread.
  const bool small = cnt <= 64;
  uint16_t* Fd = small ? S.fdst : S.lit;     // destination
  uint16_t* Fl = small ? S.flen : S.out;     // length
  uint32_t* Fp = small ? S.fpk : S.oflo;     // source | period << 16
  uint16_t* Fr = small ? S.frng : S.lst;     // dependency range within the chunk
  uint32_t md0[5], mM[5], ms[5], md[5];
  const uint32_t per = (cnt + kWG - 1) / kWG, a0 = min(cnt, t * per), a1 = min(cnt, a0 + per);
  // dependency ranges of this thread's matches (reads Fd, Fl of earlier ones)
  auto ranges = [&]() {
#pragma unroll
    for (uint32_t u = 0; u < 5; u++) {
      const uint32_t a = a0 + u;
      if (a < a1) {
        const int32_t s = (int32_t)ms[u] - 16384;
        const uint32_t w = min(md[u], mM[u]);
        uint32_t lo = a, hi = a;
        if (s + (int32_t)w > 0) {
          const uint32_t ws = s > 0 ? (uint32_t)s : 0u, we = (uint32_t)(s + (int32_t)w);
          // lo = first earlier match whose destination ends after ws, hi =
          // first whose destination starts at or after we (hi >= lo)
          uint32_t l1 = 0, h1 = a, l2 = 0, h2 = a;
          while (l1 < h1 || l2 < h2) {
            const uint32_t m1 = (l1 + h1) >> 1, m2 = (l2 + h2) >> 1;
            const uint32_t e1 = (uint32_t)Fd[min(m1, a - 1)] + Fl[min(m1, a - 1)];
            const uint32_t b2 = Fd[min(m2, a - 1)];
            if (l1 < h1) { if (e1 > ws) h1 = m1; else l1 = m1 + 1; }
            if (l2 < h2) { if (b2 >= we) h2 = m2; else l2 = m2 + 1; }
          }
          lo = l1;
          hi = l2;
        }
        const uint32_t c0 = a & ~63u;
        const uint32_t plo = max(lo, c0) - c0, phi = max(hi, c0) - c0;   // both <= 63
        Fr[a] = (uint16_t)(plo | (phi << 8));
        Fp[a] = ms[u] | (md[u] << 16);
      }
    }
  };
  if (!small) {                              // more than 64: fields packed into the tables
#pragma unroll
    for (uint32_t u = 0; u < 5; u++) {
      const uint32_t a = a0 + u;
      const uint32_t q = a < a1 ? min((uint32_t)S.lst[kMaxSeq - 1 - a], ns - 1) : 0u;
      const uint32_t L = (uint32_t)S.lit[q + 1] - S.lit[q];
      const uint32_t M = min((uint32_t)S.out[q + 1] - S.out[q] - L, blen);
      const uint32_t d0 = S.out[q] + L;
      const uint64_t of = (uint64_t)S.oflo[q] | ((uint64_t)S.ofhi[q] << 32);
      const uint64_t dabs = sb + d0;
      md0[u] = d0;
      mM[u] = M;
      // of + M > sb here (the source window touches the block) and of < dabs,
      // so the relative source fits in [-16384, 16384)
      ms[u] = (uint32_t)((int64_t)of - (int64_t)sb + 16384) & 0xFFFFu;
      md[u] = dabs > of ? (uint32_t)min<uint64_t>(dabs - of, 32767) : 1u;
    }
    __syncthreads();                         // Fd, Fl are the tables just read
#pragma unroll
    for (uint32_t u = 0; u < 5; u++) {
      const uint32_t a = a0 + u;
      if (a < a1) {
        Fd[a] = (uint16_t)md0[u];
        Fl[a] = (uint16_t)mM[u];
      }
    }
    __syncthreads();
    ranges();
    __syncthreads();
  }
  CLK_MARK(S, 6);
  // ---- stage 5: tile -> HBM by n threads, this one the i-th; through the L2,
  // to where every XCD sees it, if some block copies from this one.  Four LDS
  // reads go out together: one at a time, a wave alone took a round trip for
  // each of its 16 (or, of 8 bytes, 32) stores.
  auto store_tile = [&](uint32_t i, uint32_t n) {
    if (!dst) return;
    const uint32_t full = blen >> 4;
    const u32x4* s4 = reinterpret_cast<const u32x4*>(S.tile);
    for (uint32_t c = i; c < full; c += 4 * n) {
      u32x4 v[4] = {};
#pragma unroll
      for (uint32_t u = 0; u < 4; u++)
        if (c + u * n < full) v[u] = s4[c + u * n];
#pragma unroll
      for (uint32_t u = 0; u < 4; u++) {
        uint8_t* p = dst + 16 * (uint64_t)(c + u * n);
        if (c + u * n >= full) break;
        if (used) {
          uint64_t* q = reinterpret_cast<uint64_t*>(p);
          __hip_atomic_store(q, (uint64_t)v[u][0] | ((uint64_t)v[u][1] << 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          __hip_atomic_store(q + 1, (uint64_t)v[u][2] | ((uint64_t)v[u][3] << 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else {
          *reinterpret_cast<u32x4*>(p) = v[u];
        }
      }
    }
    for (uint32_t c = 16 * full + i; c < blen; c += n) {
      if (used) __hip_atomic_store(dst + c, S.tile[c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      else dst[c] = S.tile[c];
    }
  };
  // No workgroup barrier from here to the end of the passes: wave 0 and
  // waves 1..3 run different code.
  const bool ov = small && nb != ~0u;
  const uint64_t c4_ = CLK_NOW();
  if (wv == 0 && cnt) {
    // wave 0's passes bound this stage: it wins issue on its SIMD meanwhile
    __builtin_amdgcn_s_setprio(2);
    bool bad = false;
    // whole-wave copy of an in-block match (any length, period and source;
    // uniform arguments): a short repeating one a byte per lane, the rest in
    // longer pieces
    auto copy_match = [&](uint32_t d0, uint32_t M, int32_t s, uint32_t d) {
      if (M > 256 || d >= M || s < 0) {
        copy_long(S, A, sb, d0, M, s, d, bad);
        return;
      }
      // byte k of the match is byte k mod d of its source; k and d are below
      // 256, so (k + 1/2) / d lies at least 1/510 away from any whole number,
      // further than the float product is off
      const float rd = 1.0f / (float)d;
      uint32_t v[4];
#pragma unroll
      for (uint32_t u = 0; u < 4; u++) {
        const uint32_t k = 64 * u + lane;
        if (64 * u < M) v[u] = S.tile[(uint32_t)s + k - d * (uint32_t)(((float)k + 0.5f) * rd)];
      }
#pragma unroll
      for (uint32_t u = 0; u < 4; u++) {
        const uint32_t k = 64 * u + lane;
        if (k < M) S.tile[d0 + k] = (uint8_t)v[u];
      }
    };
    for (uint32_t c0 = 0; c0 < cnt; c0 += 64) {
      const uint32_t a = c0 + lane;
      const bool have = a < cnt;
      const uint32_t aa = have ? a : c0;
      const uint32_t pk = Fp[aa], dst = Fd[aa], len = Fl[aa];
      const int32_t s = (int32_t)(pk & 0xFFFFu) - 16384;
      const uint32_t d = (pk >> 16) & 0x7FFFu;
      uint32_t plo, phi;                      // the earlier matches of the chunk it copies from
      if (small) {
        if (!wait) near_ranges();
        plo = nlo;
        phi = nhi;
      } else {
        const uint32_t rng = Fr[aa];
        plo = rng & 63u;
        phi = (rng >> 8) & 63u;
      }
      const uint64_t needm = have && phi > plo ? (1ull << phi) - (1ull << plo) : 0ull;
      const bool fast = s >= 0 && len <= kFastLen && (d >= len || d == 1);
      const uint32_t nit = (len + 63) >> 6;   // its 64-byte pieces
      bool pending = have;
      uint64_t done = ~__ballot(pending);
      for (uint32_t pass = 0; pass < 128; pass++) {   // at least one match a pass
        const bool ready = pending && (needm & ~done) == 0;
        const uint64_t m = __ballot(ready);
        if (!m) break;
        CLK_ADD(S, 10, 1);
        uint64_t mf = __ballot(ready && fast), later = 0;
        if (mf) {
          // the ready matches' 64-byte pieces side by side, then sixteen at a
          // time, four lanes a piece, each lane 16 bytes: a pass has about ten
          // ready matches of some 20 bytes, so one lane a match (17 words read,
          // up to 64 byte stores) left most lanes idle behind the longest one
          uint32_t at = mbcnt(mf), n = (uint32_t)__popcll(mf);
          if (__ballot(ready && fast && nit > 1)) {
            at = wave_scan(ready && fast ? nit : 0u);
            later = __ballot(ready && fast && at > 64);        // no room: in the next pass
            mf &= ~later;
            n = __builtin_amdgcn_readlane(at, 63 - (uint32_t)__builtin_clzll(mf));
            at -= nit;
          }
          if (ready && fast && at + nit <= 64)
            for (uint32_t u = 0; u < nit; u++)
              S.rdy[at + u] = (uint64_t)(dst | (len << 16)) |
                              ((uint64_t)((uint32_t)s | (u << 22) | (d == 1 ? 1u << 31 : 0u)) << 32);
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
          const uint32_t sub = 16 * (lane & 3);
          for (uint32_t g0 = 0; g0 < n; g0 += 16) {
            const uint32_t i = g0 + (lane >> 2);
            const uint64_t q = S.rdy[min(i, n - 1)];
            const uint32_t L = (uint32_t)q >> 16, h = (uint32_t)(q >> 32), o = ((h >> 16) & 0xC0u) + sub;
            if (i < n && o < L) {
              // the last piece of 16 bytes or more is moved back to end with the match
              const uint32_t k = L >= 16 ? min(o, L - 16) : 0u;
              const bool one = h >> 31;       // the byte before the match, repeated
              u32x4 v = ld128(S.tile + (h & 0xFFFFu) + (one ? 0u : k));
              if (one) {
                const uint32_t x = (v[0] & 0xFFu) * 0x01010101u;
                v = u32x4{x, x, x, x};
              }
              st_upto16(S.tile + ((uint32_t)q & 0xFFFFu) + k, v, min(L, 16u));
            }
          }
        }
        uint64_t slow = __ballot(ready && !fast);
        const uint64_t c1_ = CLK_NOW();
        CLK_ADD(S, 11, __popcll(slow));
        while (slow) {                        // wave-uniform
          const uint32_t l = (uint32_t)__builtin_ctzll(slow);
          slow &= slow - 1;
          const uint32_t k = __builtin_amdgcn_readlane(pk, l);
          copy_match(__builtin_amdgcn_readlane(dst, l), __builtin_amdgcn_readlane(len, l),
                     (int32_t)(k & 0xFFFFu) - 16384, (k >> 16) & 0x7FFFu);
        }
        CLK_ADD(S, 12, CLK_NOW() - c1_);
        pending = pending && (!ready || ((later >> lane) & 1));
        done |= m & ~later;
        // the next pass reads what this one wrote (LDS operations of a wave
        // are performed in order; the fence keeps the compiler from moving
        // the reads above the stores)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      }
      if (__ballot(pending)) bad = true;      // unreachable for a valid block
    }
    if (bad) S.err = 1;
    __builtin_amdgcn_s_setprio(1);
    CLK_ADD(S, 13, CLK_NOW() - c4_);
  }
  if (wv == 0 && ov && used) {
    // others may be waiting for this block: stage 5 by wave 0 alone, while the
    // others prepare the next block
    store_tile(lane, 64);
    stores_done();
    if (lane == 0) __hip_atomic_store(A.flags + b, epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  } else if (wv != 0 && ov) {
    // the preparation has slack (it ends well before wave 0's passes): it
    // yields issue to the waves on their workgroups' critical paths
    __builtin_amdgcn_s_setprio(0);
    prep_ring(S, A, nb);
    __builtin_amdgcn_s_setprio(1);
    CLK_ADD1(S, 14, CLK_NOW() - c4_);
  }
  __syncthreads();
  const bool prepared = ov && uni(S.pok) != 0;
  CLK_ADD(S, 15, prepared ? 1 : 0);
  CLK_MARK(S, 7);
  if (S.err) {
    if (t == 0) latch(A.ctl, kStCorrupt);
    return kNext | (ov ? 0u : kUsed) | (prepared ? kPrepared : 0u);   // ov: published, if at all
  }

  // ---- stage 5, unless wave 0 has done it
  if (!(ov && used)) store_tile(t, kWG);
  CLK_MARK(S, 8);
#ifdef LZ_STAGE_CLOCKS
  if (t == 0) S.clk[9] += 1;
#endif
  return kNext | (prepared ? kPrepared : 0u) | (used && !ov ? kUsed : 0u);
}


// Once per workgroup: literal LUT image into LDS, small-stream cumulative tables.
__device__ __forceinline__ void load_tables(Smem& S, const DevArgs& A) {
  const uint32_t t = threadIdx.x, wv = uni(t >> 6);
  // the LUT image (256-byte aligned in the workspace) straight into LDS
  static_assert(kLutLit % (4 * kWG) == 0, "whole LUT rounds");
#pragma unroll 1
  for (uint32_t i = 0; i < kLutLit / (4 * kWG); i++)
    lds_dma16(A.lut + 4 * (t + kWG * i), S.lut + 4 * (64 * wv + kWG * i));
  if (t < 3 * 64) {          // waves 0..2: one table each, 4 symbols per lane
    const uint32_t k = t >> 6, lane = t & 63;
    const uint8_t* tab = A.arc + A.off_tables + 512 * (k + 1);
    uint32_t f[4], sum = 0;                          // slots, and symbols that occur << 16
    for (int q = 0; q < 4; q++) {
      f[q] = (uint32_t)tab[2 * (4 * lane + q)] | ((uint32_t)tab[2 * (4 * lane + q) + 1] << 8);
      sum += f[q] + (f[q] ? 1u << 16 : 0u);
    }
    const uint32_t incl = wave_scan(sum), all = __builtin_amdgcn_readlane(incl, 63);
    uint32_t c = incl - sum;
    for (int q = 0; q < 4; q++) {
      if (f[q]) {
        S.cum[k][c >> 16] = (uint16_t)c;
        S.sym[k][c >> 16] = (uint8_t)(4 * lane + q);
      }
      c += f[q] + (f[q] ? 1u << 16 : 0u);
    }
    for (uint32_t r = (all >> 16) + lane; r < 257; r += 64) {     // above every slot
      S.cum[k][r] = (uint16_t)all;
      if (r < 256) S.sym[k][r] = 0;
    }
  }
  vm_wait();                      // this wave's LUT rows, before the barrier
  __syncthreads();
  // bucket index of each short stream: bucket b starts at slot b << bs
  for (uint32_t e = t; e < 3 * kBuckets; e += kWG) {
    const uint32_t k = e / kBuckets, b = e % kBuckets;
    S.bkt[k][b] = (uint8_t)search_sym(S.cum[k], b << (A.P[1 + k] - 7));
  }
}

// By ticket (A.flow): one launch over the whole level-ordered queue.  A
// workgroup decodes the block of its ticket and publishes it by setting the
// block's flag to this launch's epoch.  Every block that it may have to wait
// for has a smaller ticket, held by a workgroup that runs, so the wait ends
// whatever else runs on the GPU and however few workgroups are resident.  The
// last workgroup to leave resets the tickets and makes the epoch current.
// The XCDs' L2s are not coherent with each other while a kernel runs, and
// writing back and invalidating them for each block costs more than it gives
// (256 MiB FASTQ 826 us, against 583 us with a launch per level).  So a tile
// is stored through the L2 (agent-scope stores) and its flag only after every
// wave's stores have completed (both only if some block copies from it: of a
// FASTQ a third of the blocks, of a genome a tenth); and a reader cannot hold
// an old copy of a line, as caches start a kernel without one and no line of a
// block is read before its flag is seen -- unless blocks share lines, because the output is
// not aligned to them (A.flow 2): then sources are read by agent-scope loads.
// (Tickets of two or four consecutive blocks, to take fewer, delay the blocks
// that others wait for: 64 levels 1134 us instead of 600.)
// A launch per level costs at least a block's latency (28 us) a level:
// 256 MiB FASTQ (6 levels) 498 us so and 410 us by ticket, 128 MiB genome (7)
// 405 and 262, 64 MiB FASTQ of 64 levels 1523 and 375.
// Otherwise a grid-stride slice of the queue's blocks q_begin .. q_end (one
// level).
// Jobs: up to four archives in one launch (the streams of a split container).
//
// k_code_place is never launched: it sets where k_decode<1>, which the compiler
// lays after all other kernels, begins in the code object.  The decoder is 83 KB
// of code, more than an instruction cache (64 KB for two CUs), and the same
// instructions wait more or less with their place.  Of all places tried (every
// 256 bytes of a page of 4 KB, and pages over 160 KB), those 0xe00 bytes into a
// page from 0x17e00 to 0x1ee00 are the best by far and alike: 256 MiB FASTQ 411 us,
// 128 MiB genome 259, 4096 reads 181.  0xe00 into other pages it is 433, 273
// and 208, anywhere else 433, 283 and 208.  The counters show as many
// instructions and fetches, and 10 % fewer cycles of waiting.  A change of size
// in any kernel of this file moves k_decode<1>: put it back to 0x1ce00 by the
// size here (tests/test_code_place.py tells where it is).
constexpr uint32_t kPlaceBytes = 0x8000;
__global__ void __attribute__((used)) k_code_place() {
  asm volatile(".fill %c0, 4, 0xbf800000" ::"i"(kPlaceBytes / 4));   // s_nop
}

template <uint32_t N>
struct Jobs {
  DevArgs a[N];
};

template <uint32_t N>
__global__ void __launch_bounds__(kWG, 3) k_decode(Jobs<N> J) {   // 3 waves per SIMD: at most 168 VGPRs
  __shared__ Smem S;
  uint32_t job = 0;
  if (N > 1)
    while (job + 1 < N && blockIdx.x >= J.a[job].wg0 + J.a[job].nwg) job++;
  const DevArgs& A = J.a[N > 1 ? job : 0];
  const uint32_t wg = blockIdx.x - A.wg0;
  // issue priority: 1 by default, 2 for wave 0's in-block passes, 0 for the
  // next block's preparation by waves 1..3 (the one stage with slack)
  __builtin_amdgcn_s_setprio(1);
  const uint32_t t = threadIdx.x;
  uint32_t qb = A.q_begin, qe = A.q_end;
  if (A.qptr) {
    qb = A.qptr[A.q_begin];
    qe = A.qptr[A.q_end];
  }
  const uint32_t total = qe - qb;
  if (wg >= total) return;                 // more workgroups than blocks
  if (A.flow && t == 0) S.nit = take_ticket(A);
#ifdef LZ_STAGE_CLOCKS
  if (t < kClkSlots) S.clk[t] = 0;
#endif
  const uint32_t epoch = A.flow ? A.ctl[kCtlEpoch] + 1 : 0u;
  load_tables(S, A);
  __syncthreads();
  uint32_t it = A.flow ? uni(S.nit) : wg;
  uint32_t b = it < total ? A.queue[qb + it] : 0u;
  bool prepared = false;      // the block's stages 0 and 1 are done
  while (it < total) {
    if (!prepared) prep_tile(S, A, b);
    const uint32_t r = decode_block(S, A, b, qb, total, it, epoch);
    const bool publish = A.flow && (r & kUsed) && uni(S.used);   // S.used is still this block's
    if (publish) stores_done();
    __syncthreads();
    if (publish && t == 0) {
      __hip_atomic_store(A.flags + b, epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    prepared = (r & kPrepared) != 0;
    if (r & kNext) {
      it = uni(S.nit);
      b = uni(S.nb);
    } else {                               // corrupt block: no ticket was taken
      if (t == 0) S.nit = A.flow ? take_ticket(A) : it + A.nwg;
      __syncthreads();
      it = uni(S.nit);
      b = it < total ? A.queue[qb + it] : 0u;
      __syncthreads();
    }
  }
  if (A.flow && t == 0) {
    const uint32_t left = __hip_atomic_fetch_add(A.ctl + kCtlLeft, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (left + 1 == min(A.nwg, total)) {
      A.ctl[kCtlTicket] = 0;
      A.ctl[kCtlLeft] = 0;
      A.ctl[kCtlEpoch] = epoch < kMaxEpoch ? epoch : 0u;
    }
  }
#ifdef LZ_STAGE_CLOCKS
  __syncthreads();
  if (t < kClkSlots) atomicAdd(reinterpret_cast<unsigned long long*>(A.ctl + kCtlClock) + t,
                               (unsigned long long)S.clk[t]);
#endif
}

// ---- setup kernels ---------------------------------------------------------

// Whether every block's dependency list names every earlier block that its
// matches copy from: decoding by ticket waits for the listed blocks alone.
// The lists can be checked against each other on the host, but not against the
// matches, so this prepares each block as the decoder does (its short streams
// hold the matches) and looks the sources up; one that is missing sets
// *unlisted.  Blocks with corrupt records are left to the decoder, which
// refuses them.  About a third of a decode, once per lz_open: 133 MB FASTQ in
// 8,116 blocks 81 us, which makes its lz_open 760 us instead of 683.
__global__ void __launch_bounds__(kWG, 3) k_check_deps(DevArgs A, uint32_t n_blocks, uint32_t* unlisted) {
  __shared__ Smem S;
  load_tables(S, A);
  __syncthreads();
  for (uint32_t b = blockIdx.x; b < n_blocks; b += gridDim.x) {
    prep_tile(S, A, b);
    if (S.pok && !(S.perr[0] | S.perr[1] | S.perr[2])) {
      const uint64_t sb = (uint64_t)b << A.bl;
      const uint64_t d0 = ld64(A.arc + A.off_dep_ptr + 8ull * b), d1 = ld64(A.arc + A.off_dep_ptr + 8ull * b + 8);
      bool missing = false;
      for (uint32_t j = threadIdx.x; j < S.pdir[2]; j += kWG) {
        const uint64_t of = (uint64_t)S.oflo[j] | ((uint64_t)S.ofhi[j] << 32), ml = S.out[j];
        if (!ml || of >= sb) continue;
        for (uint64_t a = of >> A.bl; a <= (min(of + ml, sb) - 1) >> A.bl; a++) {
          uint64_t lo = d0, hi = d1;                    // first listed block that is a or later
          while (lo < hi) {
            const uint64_t mid = (lo + hi) >> 1;
            if (ld32(A.arc + A.off_dep_idx + 4 * mid) < a) lo = mid + 1; else hi = mid;
          }
          missing |= lo == d1 || ld32(A.arc + A.off_dep_idx + 4 * lo) != a;
        }
      }
      if (missing) *unlisted = 1;
    }
    __syncthreads();                                    // the tables are read no more
  }
}

// Packed literal decode entry of slot u: symbol | f << 8 | (u - c_s) << 20.
__global__ void k_build_lut(const uint8_t* arc, uint64_t off_tables, uint32_t P, uint32_t* lut) {
  __shared__ uint32_t cum[257];
  __shared__ uint32_t fr[256];
  for (int s = threadIdx.x; s < 256; s += blockDim.x)
    fr[s] = (uint32_t)arc[off_tables + 2 * s] | ((uint32_t)arc[off_tables + 2 * s + 1] << 8);
  __syncthreads();
  if (threadIdx.x == 0) {
    cum[0] = 0;
    for (int s = 0; s < 256; s++) cum[s + 1] = cum[s] + fr[s];
  }
  __syncthreads();
  const uint32_t M = 1u << P;
  for (uint32_t u = threadIdx.x; u < kLutLit; u += blockDim.x) {
    if (cum[256] != M || u >= M) { lut[u] = 0; continue; }
    uint32_t lo = 0;
    for (uint32_t step = 128; step; step >>= 1)
      if (cum[lo + step] <= u) lo += step;
    lut[u] = lo | ((fr[lo] & 0xFFFu) << 8) | ((u - cum[lo]) << 20);
  }
}

__global__ void k_fill_u32(uint32_t* p, uint64_t n, uint32_t v) {
  for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x) p[i] = v;
}

__global__ void k_fill_u64(uint64_t* p, uint64_t n, uint64_t v) {
  for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x) p[i] = v;
}

}  // namespace

// ---- host launchers (called from runtime.cpp) -------------------------------

size_t lz_decode_smem_bytes() { return sizeof(Smem); }

static DevArgs make_args(const lz_handle* h) {
  DevArgs A{};
  const ArchiveView& v = h->av;
  A.arc = v.base;
  A.n = v.n;
  A.off_tables = v.off_tables;
  A.off_dir = v.off_dir;
  A.off_dep_ptr = v.off_dep_ptr;
  A.off_dep_idx = v.off_dep_idx;
  A.off_payload = v.off_payload;
  A.bl = v.block_log2;
  A.w = v.offset_width;
  A.m = v.min_match;
  A.lit_lanes = v.lit_lanes;
  A.seq_lanes = v.seq_lanes;
  for (int k = 0; k < 4; k++) A.P[k] = v.prob_bits[k];
  A.lut = h->ws.lut;
  A.flags = h->ws.flags;
  A.ctl = h->ws.ctl;
  // A wait of the decoder ends by itself unless the archive was changed after
  // lz_open; 2^20 polls are about a second, so no less than that: a limit that
  // the caller set for the planner's waits must not fail a valid decode.
  A.spin_limit = std::max(h->tune.spin_limit, 1u << 20);
  return A;
}

static int launch_ok(const char* what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return lz_fail(LZ_EDEVICE, "%s: %s", what, hipGetErrorString(e));
  return LZ_OK;
}

static uint32_t decode_slots(const lz_handle* h) { return (uint32_t)(h->n_cu * std::max(1u, h->tune.wg_per_cu)); }

int lz_launch_setup(lz_handle* h, hipStream_t s) {
  const ArchiveView& v = h->av;
  hipLaunchKernelGGL(k_build_lut, dim3(1), dim3(256), 0, s, v.base, v.off_tables, v.prob_bits[0], h->ws.lut);
  const uint64_t nb = v.n_blocks;
  const uint32_t grid = (uint32_t)std::min<uint64_t>(4096, (nb + 255) / 256 + 1);
  hipLaunchKernelGGL(k_fill_u32, dim3(grid), dim3(256), 0, s, h->ws.mark, nb, 0u);
  hipLaunchKernelGGL(k_fill_u64, dim3(grid), dim3(256), 0, s, h->ws.addr, nb, 0ull);
  // k_closure takes a list entry as pushed once its upper half is the call's
  // epoch (1, 2, ...): what the caller's memory held before must not look so
  hipLaunchKernelGGL(k_fill_u64, dim3(grid), dim3(256), 0, s, h->ws.list, nb, 0ull);
  hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(64), 0, s, h->ws.ctl, (uint64_t)kCtlWords, 0u);
  return launch_ok("lz_open setup kernels");
}

// After lz_launch_setup: ctl[kCtlUnlisted] is set if a dependency list is not
// complete (and the status word, if a block is corrupt: the caller clears the
// control words again).
int lz_launch_check_deps(lz_handle* h, hipStream_t s) {
  const uint32_t nb = (uint32_t)h->av.n_blocks;
  hipLaunchKernelGGL(k_check_deps, dim3(std::min(nb, decode_slots(h))), dim3(kWG), 0, s, make_args(h), nb,
                     h->ws.ctl + kCtlUnlisted);
  return launch_ok("lz_open dependency check");
}

int lz_launch_clear_ctl(lz_handle* h, hipStream_t s) {
  hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(64), 0, s, h->ws.ctl, (uint64_t)kCtlWords, 0u);
  return launch_ok("lz_open control words");
}

// Whether the blocks of a by-ticket launch have their cache lines (128 bytes)
// to themselves (1) or share some (2): see k_decode.  `at`: an address that
// every block's output lies a multiple of the block size from.
static uint32_t flow_mode(const DevArgs& A, uint64_t at) {
  return A.bl >= 7 && (at & 127) == 0 ? 1u : 2u;
}

// One archive on the first nwg workgroups.
static void launch_decode(DevArgs A, uint32_t nwg, hipStream_t s) {
  A.wg0 = 0;
  A.nwg = nwg;
  hipLaunchKernelGGL(k_decode<1>, dim3(nwg), dim3(kWG), 0, s, Jobs<1>{{A}});
}

// The whole file in one launch: by ticket, or, of one level, where nothing
// waits and tickets are all overhead, in static slices (32 MiB of noise,
// stored blocks: 112 us by ticket, 68 us in slices, before those blocks were
// copied in one step; 27 us in slices since).
static DevArgs whole_file(const lz_handle* h, uint8_t* out) {
  DevArgs A = make_args(h);
  A.queue = h->ws.queue;
  A.out = out;
  A.flow = h->av.n_levels > 1 ? flow_mode(A, reinterpret_cast<uintptr_t>(out)) : 0u;
  A.q_end = (uint32_t)h->av.n_blocks;
  return A;
}

// By ticket only what every block waits for is known to be complete; a level
// at a time, a source in a lower level is there whether it is listed or not.
static bool one_launch(const lz_handle* h) { return h->tune.sync_mode == 0 && h->deps_listed; }

// Whether that many blocks of the archive are decoded faster a level at a time.
// By ticket every block costs three updates of counters that all workgroups
// share (about 85 in a microsecond), and every level but the first one is
// hidden; a launch per level costs a block's latency each, the less the smaller
// the blocks.  So few levels of many small blocks are left to launches of their
// own, those of more blocks than workgroups run at once.  Measured by ticket
// and per level: 8 MB FASTQ of 1 KiB blocks in 2 levels 159 and 126 us, in 4
// 163 and 156, in 5 158 and 160; of 2 KiB in 3 108 and 90, in 4 110 and 103
// (a genome 112 and 142); of 8 KiB in 2 74 and 53, in 3 78 and 72 (a genome
// 93 and 114); 508 blocks of 16 KiB in 2 51 and 55.
static bool few_levels(const lz_handle* h) {
  const uint32_t bl = h->av.block_log2;
  return h->av.n_levels <= (bl <= 10 ? 4u : bl == 11 ? 3u : bl <= 13 ? 2u : 1u);
}
static bool shallow(const lz_handle* h, uint64_t blocks) { return few_levels(h) && blocks > decode_slots(h); }

int lz_launch_decode_all(lz_handle* h, uint8_t* out, hipStream_t s) {
  DevArgs A = whole_file(h, out);
  const uint32_t slots = decode_slots(h);
  if (one_launch(h) && !shallow(h, h->av.n_blocks)) {
    launch_decode(A, std::min(A.q_end, slots), s);
    return launch_ok("lz_decode_all");
  }
  A.flow = 0;
  uint32_t base = 0;
  for (uint32_t L = 0; L < h->av.n_levels; L++) {
    const uint32_t c = h->level_count[L];
    if (c) {
      A.q_begin = base;
      A.q_end = base + c;
      launch_decode(A, std::min(c, slots), s);
    }
    base += c;
  }
  return launch_ok("lz_decode_all");
}

// Whether n archives are decoded at once (below): all by ticket, and not all of
// few levels with one that is faster a level at a time: then one after the other
// (streams of an 8 MB FASTQ in 1 KiB blocks of 2 levels 254 us at once and
// 208 one by one, of 4 levels 267 and 261; of up to 32 levels 226 and 318).
bool lz_decode_together(lz_handle* const* h, uint32_t n) {
  bool all_few = true, any_shallow = false;
  for (uint32_t k = 0; k < n; k++) {
    if (!one_launch(h[k])) return false;
    all_few &= few_levels(h[k]);
    any_shallow |= h[k]->av.n_levels > 1 && shallow(h[k], h[k]->av.n_blocks);
  }
  return !(all_few && any_shallow);
}

// Whole-file decodes of n <= 4 non-empty archives at once, out[k] the output
// of h[k].  Every archive gets the workgroups that it would have alone, the
// shortest archive first (a chain of levels, or a few slow blocks, is best
// begun at once): as many as fit run, and as an archive's end, the next one's
// take their places, so the chip stays full whatever a block of each costs.
// (With the resident workgroups shared out by blocks, the 350 blocks of a
// 64 MiB FASTQ's id lines, 50 us each, took 300 us on their 65.)  One after
// the other the four streams took 51 + 91 + 124 + 98 us, 124 for the 25
// blocks and as many levels of the '+' lines.
int lz_launch_decode_many(lz_handle* const* h, uint8_t* const* out, uint32_t n, hipStream_t s) {
  Jobs<4> J{};
  uint32_t at[4], m = 0;
  for (uint32_t k = 0; k < n; k++) {
    uint32_t i = m++;
    for (; i && h[at[i - 1]]->av.n_blocks > h[k]->av.n_blocks; i--) at[i] = at[i - 1];
    at[i] = k;
  }
  uint32_t wg = 0;
  for (uint32_t k = 0; k < m; k++) {
    const lz_handle* a = h[at[k]];
    J.a[k] = whole_file(a, out[at[k]]);
    J.a[k].wg0 = wg;
    J.a[k].nwg = (uint32_t)std::min<uint64_t>(a->av.n_blocks, decode_slots(a));
    wg += J.a[k].nwg;
  }
  for (uint32_t k = m; k < 4; k++) J.a[k].wg0 = wg;      // no workgroups
  if (wg) hipLaunchKernelGGL(k_decode<4>, dim3(wg), dim3(kWG), 0, s, J);
  return launch_ok("lz_split_decode_all");
}

// ---- verification: per-block FNV-1a-64 against the directory -----------------
//
// h' = (h ^ byte) p is a serial chain over the bytes, but only through the low
// 8 bits of h: with l the low byte, h ^ byte = h + d, d = (l ^ byte) - l, so
//   h_n = h_0 p^n + sum of d_i p^(n-i)    (mod 2^64),
// a sum that segments of the data contribute to independently once the low
// byte at each segment's start is known.  The low byte's own recurrence
// l' = (l ^ byte) 0xb3 mod 256 carries no bit downwards, and bit k of l enters
// bit k of l' by xor alone (0xb3 is odd).  So the bits are resolved from the
// lowest: with the bits below k known at every segment's start, a pass over
// the segment from a start with bit k zero gives the bit the segment xors into
// bit k, and a prefix xor over the segments (a ballot) gives bit k at every
// start.  Bit 0 is the parity of the bytes' bits 0; seven passes of one
// instruction a byte (two a pair, two half segments in one packed 16-bit
// register) replace the rest of the chain, and one more gives the d, summed up
// with their weights by dot products.
// 128 MiB in 8192 blocks, blocks and hash over the hashes together: 71 us (57
// and 16); with the chain in one thread per block (292 us) and one thread for
// the hash over the hashes (1353 us) it was 1716 us.  Bound by the passes'
// instructions, not by memory (27 us at a copy's rate).
namespace {

constexpr uint32_t kSeg = 64;                    // bytes of a lane's segment
constexpr uint32_t kChunk = 64 * kSeg;           // bytes a wave takes at once

constexpr uint64_t fnv_pow(uint32_t n) {
  uint64_t r = 1, q = kFnvPrime;
  for (; n; n >>= 1, q *= q)
    if (n & 1) r *= q;
  return r;
}
__device__ __forceinline__ uint64_t fnv_pow_at(uint32_t n) {      // n <= kChunk
  uint64_t r = 1, q = kFnvPrime;
#pragma unroll 1
  for (uint32_t s = 0; s < 13; s++) {
    r = n & (1u << s) ? r * q : r;
    q *= q;
  }
  return r;
}

typedef uint16_t u16x2 __attribute__((vector_size(4)));
typedef int16_t s16x2 __attribute__((vector_size(4)));

// A full segment's sum: bytes i and 32 + i (i < 32) contribute their d with the
// weights p^(64 - i) and p^(32 - i).  The weights are split into four signed
// 16-bit digits, so that two-element dot products add both: a digit's sum
// stays below 64 * 255 * 2^15 < 2^31.
struct FnvWeights {
  uint32_t w[4][kSeg / 2];         // digit k of both weights, packed
};
constexpr FnvWeights fnv_weights() {
  FnvWeights f = {};
  for (uint32_t i = 0; i < kSeg / 2; i++)
    for (uint32_t h = 0; h < 2; h++) {
      uint64_t v = fnv_pow(kSeg - kSeg / 2 * h - i);
      for (uint32_t k = 0; k < 4; k++) {
        f.w[k][i] |= (uint32_t)(v & 0xFFFFu) << (16 * h);
        v = (v >> 16) + ((v >> 15) & 1u);        // the digit was taken as signed
      }
    }
  return f;
}

// Bit k of the low byte at the halves' starts (sa, sb), from the bits xa, xb
// that the halves xor into it and the bit c before the round; c becomes the
// bit after it.
template <uint32_t NW>
__device__ __forceinline__ void fnv_bit(uint32_t k, uint32_t xa, uint32_t xb, uint32_t& c, uint32_t& sa, uint32_t& sb,
                                        uint32_t wv, uint32_t (*bits)[8]) {
  const uint64_t x = __ballot(xa ^ xb);
  uint32_t all = (uint32_t)__popcll(x), before = c;
  if (NW > 1) {
    if (lane_id() == 0) bits[wv][k] = all & 1u;
    __syncthreads();
    all = 0;
    for (uint32_t q = 0; q < NW; q++) {
      const uint32_t b = bits[q][k];
      all ^= b;
      before ^= q < wv ? b : 0u;
    }
  }
  const uint32_t ka = (mbcnt(x) ^ before) & 1u;
  sa |= ka << k;
  sb |= (ka ^ xa) << k;
  c = (c ^ all) & 1u;
}

// The sum that this lane's segment contributes at its end, the 64 bytes at p
// (have: it has one; p is not read else).  low: the low byte of the hash before
// the round, then after it.
template <uint32_t NW>
__device__ __forceinline__ uint64_t fnv_segment(const uint8_t* p, bool have, uint32_t& low, uint32_t wv,
                                                uint32_t (*bits)[8]) {
  constexpr FnvWeights kW = fnv_weights();
  uint32_t w[kSeg / 4] = {};
  if (have) {
#pragma unroll
    for (uint32_t q = 0; q < kSeg / 16; q++) {
      const u32x4 v = ld128(p + 16 * q);
#pragma unroll
      for (uint32_t r = 0; r < 4; r++) w[4 * q + r] = v[r];
    }
  }
  // byte i of the first half segment with byte i of the second
  u16x2 pr[kSeg / 2];
#pragma unroll
  for (uint32_t i = 0; i < kSeg / 2; i++)
    pr[i] = (u16x2)__builtin_amdgcn_perm(w[kSeg / 8 + i / 4], w[i / 4], 0x0C040C00u + 0x00010001u * (i % 4));
  // bit 0: the parity of the bytes' bits 0
  uint32_t xa = 0, xb = 0, sa = 0, sb = 0, next = low & 1u;
#pragma unroll
  for (uint32_t q = 0; q < kSeg / 8; q++) {
    xa ^= w[q];
    xb ^= w[kSeg / 8 + q];
  }
  xa = __builtin_popcount(xa & 0x01010101u) & 1u;
  xb = __builtin_popcount(xb & 0x01010101u) & 1u;
  fnv_bit<NW>(0, xa, xb, next, sa, sb, wv, bits);
  const uint32_t mine = have ? 1u : 0u;
#pragma unroll 1
  for (uint32_t k = 1; k < 8; k++) {
    u16x2 l = {(uint16_t)sa, (uint16_t)sb};
#pragma unroll
    for (uint32_t i = 0; i < kSeg / 2; i++) l = (l ^ pr[i]) * (uint16_t)0xb3;
    uint32_t c = (low >> k) & 1u;
    fnv_bit<NW>(k, ((uint32_t)l[0] >> k) & mine, ((uint32_t)l[1] >> k) & mine, c, sa, sb, wv, bits);
    next |= c << k;
  }
  low = next;
  // d = (l ^ byte) - l (the bits of l above its low byte cancel)
  u16x2 l = {(uint16_t)sa, (uint16_t)sb};
  int32_t acc[4] = {0, 0, 0, 0};
#pragma unroll
  for (uint32_t i = 0; i < kSeg / 2; i++) {
    const u16x2 x = l ^ pr[i], d = x - l;
    l = x * (uint16_t)0xb3;
#pragma unroll
    for (uint32_t k = 0; k < 4; k++) {
      const s16x2 c = {(int16_t)(kW.w[k][i] & 0xFFFFu), (int16_t)(kW.w[k][i] >> 16)};
      acc[k] = __builtin_amdgcn_sdot2((s16x2)d, c, acc[k], false);
    }
  }
  const uint64_t sum = (uint64_t)(int64_t)acc[0] + ((uint64_t)(int64_t)acc[1] << 16) +
                       ((uint64_t)(int64_t)acc[2] << 32) + ((uint64_t)(int64_t)acc[3] << 48);
  return have ? sum : 0;
}

// A workgroup of NW waves extends the hash h by the n bytes at p, kChunk * NW
// bytes a round (NW = 1: each wave on its own bytes, no barrier).  Every lane
// returns the hash.  Whole rounds only carry the low byte from one to the
// next: each lane's sums are weighted and added up over the rounds, and the
// lanes put together once at the end.  Then a round of the whole segments that
// are left, and the last bytes (less than a segment) one by one.
template <uint32_t NW>
__device__ uint64_t fnv_extend(uint64_t h, const uint8_t* p, uint64_t n, uint64_t (*part)[2], uint32_t (*bits)[8]) {
  const uint32_t lane = lane_id(), wv = NW > 1 ? uni(threadIdx.x >> 6) : 0u;
  const uint32_t o = wv * kChunk + lane * kSeg;                   // this lane's segment
  uint64_t at = 0, T = 0;
  uint32_t low = (uint32_t)h & 0xFFu;
  for (; at + kChunk * NW <= n; at += kChunk * NW) {
    T = T * fnv_pow(kChunk * NW) + fnv_segment<NW>(p + at + o, true, low, wv, bits);
    h *= fnv_pow(kChunk * NW);
  }
  if (at) {
#pragma unroll
    for (uint32_t s = 0; s < 6; s++) {                            // lane 0: the wave's sum
      const uint64_t right = __shfl(T, (int)(lane + (1u << s)) & 63);
      T = T * fnv_pow(kSeg << s) + right;
    }
    if (NW == 1) {
      h += __shfl(T, 0);
    } else {
      if (lane == 0) part[wv][0] = T;
      __syncthreads();
      uint64_t sum = 0;
#pragma unroll 1
      for (uint32_t q = 0; q < NW; q++) sum = sum * fnv_pow(kChunk) + part[q][0];
      h += sum;
      __syncthreads();
    }
  }
  const uint32_t todo = (uint32_t)(n - at) & ~(kSeg - 1);         // whole segments, less than a round
  if (todo) {
    const uint32_t end = min(todo, (wv + 1) * kChunk);            // of the wave's bytes
    const bool have = o < todo;
    uint64_t R = fnv_segment<NW>(p + at + o, have, low, wv, bits);
    R *= fnv_pow_at(have ? end - o - kSeg : 0u);
    for (uint32_t s = 32; s; s >>= 1) R += __shfl(R, (int)(lane + s) & 63);
    const uint32_t len = wv * kChunk < todo ? end - wv * kChunk : 0u;
    if (NW == 1) {
      h = h * fnv_pow_at(len) + __shfl(R, 0);
    } else {
      if (lane == 0) {
        part[wv][0] = R;
        part[wv][1] = fnv_pow_at(len);
      }
      __syncthreads();
#pragma unroll 1
      for (uint32_t q = 0; q < NW; q++) h = h * part[q][1] + part[q][0];
      __syncthreads();
    }
    at += todo;
  }
  const uint32_t left = (uint32_t)(n - at);                       // less than a segment
  const uint32_t v = lane < left ? p[at + lane] : 0u;
#pragma unroll 1
  for (uint32_t i = 0; i < left; i++) h = (h ^ __builtin_amdgcn_readlane(v, i)) * kFnvPrime;
  return h;
}

// Blocks b0 .. b0 + nb - 1 of the file, decoded at out (block b0 first): one
// wave per block hashes it, and the hash is compared with the directory's.
__global__ void __launch_bounds__(256) k_fnv_blocks(const uint8_t* arc, uint64_t off_dir, const uint8_t* out, uint64_t n,
                                                    uint32_t bl, uint64_t b0, uint64_t nb, uint64_t* hashes,
                                                    uint32_t* ctl) {
  const uint64_t i = (uint64_t)blockIdx.x * 4 + uni(threadIdx.x >> 6);
  if (i >= nb) return;
  const uint64_t b = b0 + i, sb = b << bl, B = 1ull << bl;
  const uint64_t h = fnv_extend<1>(kFnvBasis, out + (i << bl), sb + B <= n ? B : n - sb, nullptr, nullptr);
  if (lane_id() == 0) {
    hashes[i] = h;
    if (h != ld64(arc + off_dir + b * kDirEntry + 24)) latch(ctl, kStHash);
  }
}

// The same for blocks of less than a wave's chunk: one thread per block.
__global__ void k_fnv_small(const uint8_t* arc, uint64_t off_dir, const uint8_t* out, uint64_t n,
                            uint32_t bl, uint64_t b0, uint64_t nb, uint64_t* hashes, uint32_t* ctl) {
  const uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x;
  if (i >= nb) return;
  const uint64_t b = b0 + i;
  const uint64_t sb = b << bl, B = 1ull << bl;
  const uint64_t len = sb + B <= n ? B : n - sb;
  const uint8_t* src = out + (i << bl);
  uint64_t h = kFnvBasis;
  const uint4* p = reinterpret_cast<const uint4*>(src);
  uint64_t k = 0;
  for (; k + 16 <= len; k += 16) {
    const uint4 v = p[k >> 4];
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int q = 0; q < 4; q++)
#pragma unroll
      for (int j = 0; j < 4; j++) h = (h ^ ((w[q] >> (8 * j)) & 0xFFu)) * kFnvPrime;
  }
  for (; k < len; k++) h = (h ^ src[k]) * kFnvPrime;
  hashes[i] = h;
  if (h != ld64(arc + off_dir + b * kDirEntry + 24)) latch(ctl, kStHash);
}

// The hash over the block hashes, one workgroup: 8192 hashes a round.
constexpr uint32_t kTreeWaves = 16;
__global__ void __launch_bounds__(64 * kTreeWaves) k_fnv_tree(const uint64_t* hashes, uint64_t nb, uint64_t* tree) {
  __shared__ uint64_t part[kTreeWaves][2];
  __shared__ uint32_t bits[kTreeWaves][8];
  const uint64_t h = fnv_extend<kTreeWaves>(kFnvBasis, reinterpret_cast<const uint8_t*>(hashes), 8 * nb, part, bits);
  if (threadIdx.x == 0) *tree = h;
}

}  // namespace

int lz_launch_verify(lz_handle* h, const uint8_t* d_out, uint64_t b0, uint64_t nb, uint64_t* d_tree,
                     void* scratch, hipStream_t s) {
  uint64_t* hashes = reinterpret_cast<uint64_t*>(scratch);
  if (nb) {
    if ((uintptr_t)d_out & 15) return lz_fail(LZ_EINVAL, "lz_verify: output must be 16-byte aligned");
    // a wave needs a whole chunk of bytes to be worth its passes
    if ((1u << h->av.block_log2) >= kChunk)
      hipLaunchKernelGGL(k_fnv_blocks, dim3((uint32_t)((nb + 3) / 4)), dim3(256), 0, s, h->av.base,
                         h->av.off_dir, d_out, h->av.n, h->av.block_log2, b0, nb, hashes, h->ws.ctl);
    else
      hipLaunchKernelGGL(k_fnv_small, dim3((uint32_t)((nb + 255) / 256)), dim3(256), 0, s, h->av.base,
                         h->av.off_dir, d_out, h->av.n, h->av.block_log2, b0, nb, hashes, h->ws.ctl);
  }
  if (d_tree) hipLaunchKernelGGL(k_fnv_tree, dim3(1), dim3(64 * kTreeWaves), 0, s, hashes, nb, d_tree);
  return launch_ok("lz_verify");
}

// ---- FASTA regions: bases of a sequence gathered from its decoded bytes -------
namespace {

// out[i] = base start + i of a sequence whose first base is at byte `offset`
// of the file, W bases per line of LB bytes; tmp holds the file bytes from
// `first` on.
__global__ void k_region_gather(const uint8_t* tmp, uint64_t first, uint64_t offset, uint64_t start,
                                uint64_t nb, uint32_t W, uint32_t LB, uint8_t* out) {
  for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < nb;
       i += (uint64_t)gridDim.x * blockDim.x) {
    const uint64_t k = start + i;
    out[i] = tmp[offset + (k / W) * LB + k % W - first];
  }
}

}  // namespace

int lz_launch_region_gather(const uint8_t* tmp, uint64_t first, uint64_t offset, uint64_t start,
                            uint64_t nb, uint32_t W, uint32_t LB, uint8_t* out, hipStream_t s) {
  const uint32_t grid = (uint32_t)std::min<uint64_t>(4096, (nb + 255) / 256);
  hipLaunchKernelGGL(k_region_gather, dim3(grid), dim3(256), 0, s, tmp, first, offset, start, nb, W, LB, out);
  return launch_ok("lz_decode_region");
}

// ---- requests: ranges, read lookups, batches --------------------------------
//
// A batch is resolved by a fixed sequence of launches whose sizes are read on
// the device, so the sequence can be captured once and replayed:
//   begin   new request and completion epochs, counters cleared
//   spans   request -> [start, end) bytes (read id through the read index)
//   scan    exclusive prefix of lengths (output offsets) and of covering-block
//           counts (request, block) pairs; capacity check
//   mark    every covering block marked with the epoch and pushed on a list
//   closure worklist over the dependency lists: each pushed block pushes its
//           unmarked dependencies (transitive closure)
//   levels  counting sort of the closure by dependency level; each block gets
//           an address: straight into the output when it lies wholly inside an
//           aligned single range, else a scratch slot
//   decode  k_decode over the level-ordered closure (same body as whole-file)
//   gather  requested bytes of scratch-resident blocks copied to the output
namespace {

struct ReqArgs {
  const uint8_t* arc;
  uint64_t n, n_blocks, off_dir, off_dep_ptr, off_dep_idx, off_ridx, n_reads;
  uint32_t bl, mode, direct, lmark;
  uint64_t a0, b0;            // mode 0: the single range
  const int64_t* ids;         // mode 1: read ids
  const lz_request* reqs;     // mode 2: requests
  const uint32_t* d_n;        // mode 2: device request count
  uint64_t n_max;
  uint8_t* out;
  uint64_t cap;
  uint64_t* offsets;          // caller's offsets (n + 1) or null
  uint64_t* spans;            // scratch: 2 per request
  uint64_t* cnt_ptr;          // scratch: n + 1
  uint64_t* offs;             // scratch: n + 1
  uint8_t* slots;
  uint64_t max_slots;
  uint32_t* mark;
  uint32_t* flags;
  uint64_t* addr;
  uint32_t* rqueue;
  uint32_t* rlevel_ptr;
  uint64_t* list;
  uint32_t* ctl;
};

__device__ __forceinline__ uint64_t* ctl64(uint32_t* ctl, uint32_t w) { return reinterpret_cast<uint64_t*>(ctl + w); }

__device__ __forceinline__ uint32_t aload(const uint32_t* p) {
  return __hip_atomic_load(const_cast<uint32_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// largest j in [0, n) with v[j] <= g (v nondecreasing, v[0] = 0)
__device__ __forceinline__ uint32_t find_req(const uint64_t* v, uint32_t n, uint64_t g) {
  uint32_t lo = 0, hi = n;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (v[mid] <= g) lo = mid; else hi = mid;
  }
  return lo;
}

// Mark block b with the request epoch; push it on the closure list if this
// call marked it first.
__device__ __forceinline__ void mark_push(const ReqArgs& R, uint32_t b, uint32_t epoch) {
  const uint32_t old = __hip_atomic_fetch_max(R.mark + b, epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (old >= epoch) return;
  const uint32_t i = __hip_atomic_fetch_add(R.ctl + kCtlListTail, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(R.list + i, ((uint64_t)epoch << 32) | b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The decode epochs near their end (one workgroup): flags of any earlier epoch
// are cleared, so that none is met again after the epochs have started over;
// true if so, and the caller resets the epoch after a barrier.  Whole-file
// decodes need no such care: each sets every flag that is ever set.
__device__ __forceinline__ bool renew_flags(const ReqArgs& R) {
  if (R.ctl[kCtlEpoch] < kRenewEpoch) return false;
  for (uint64_t i = threadIdx.x; i < R.n_blocks; i += blockDim.x)
    if (R.flags[i] != kFlagLeaf) R.flags[i] = 0;
  return true;
}

// One workgroup.  First the address-table entries of the previous call's
// closure (still in the work list) are cleared, so that afterwards exactly the
// blocks of this call's closure have an address: a match whose source lies in
// any other block reads a null entry and fails as corrupt instead of following
// a pointer into a buffer of an earlier call.  Then the counters are reset.
__global__ void __launch_bounds__(256) k_req_begin(ReqArgs R) {
  const uint32_t t = threadIdx.x;
  const uint32_t prev = min(R.ctl[kCtlListTail], (uint32_t)R.n_blocks);
  for (uint32_t i = t; i < prev; i += blockDim.x) {
    const uint32_t b = (uint32_t)R.list[i];
    if (b < R.n_blocks) R.addr[b] = 0;
  }
  const bool renew = renew_flags(R);
  __syncthreads();
  if (t < 64) R.ctl[kCtlLevelCnt + t] = 0;
  if (t == 0) {
    if (renew) R.ctl[kCtlEpoch] = 0;
    R.ctl[kCtlREpoch] += 1;
    R.ctl[kCtlListTail] = 0;
    R.ctl[kCtlListHead] = 0;
    R.ctl[kCtlListDone] = 0;
    R.ctl[kCtlSlots] = 0;
    uint64_t n = R.n_max;
    if (R.mode == 2) n = min((uint64_t)*R.d_n, R.n_max);
    R.ctl[kCtlNReq] = (uint32_t)n;
    *ctl64(R.ctl, kCtlTotal) = 0;
    *ctl64(R.ctl, kCtlPairs) = 0;
  }
}

__device__ __forceinline__ bool read_span(const ReqArgs& R, int64_t r, uint64_t& s, uint64_t& e) {
  if (!R.off_ridx || r < 0 || (uint64_t)r >= R.n_reads) return false;
  s = ld64(R.arc + R.off_ridx + 8ull * (uint64_t)r);
  e = ld64(R.arc + R.off_ridx + 8ull * (uint64_t)r + 8);
  return true;
}

__global__ void k_req_spans(ReqArgs R) {
  const uint32_t nreq = R.ctl[kCtlNReq];
  for (uint32_t j = blockIdx.x * blockDim.x + threadIdx.x; j < nreq; j += gridDim.x * blockDim.x) {
    uint64_t s = 0, e = 0;
    bool ok = true;
    if (R.mode == 0) {
      s = R.a0;
      e = R.a0 + R.b0;
    } else if (R.mode == 1) {
      ok = read_span(R, R.ids[j], s, e);
    } else {
      const lz_request q = R.reqs[j];
      if (q.kind == 0) {
        ok = read_span(R, q.a, s, e);
      } else if (q.kind == 1 && q.a >= 0 && q.b >= 0 && (uint64_t)q.a <= R.n && (uint64_t)q.b <= R.n - (uint64_t)q.a) {
        s = (uint64_t)q.a;
        e = s + (uint64_t)q.b;
      } else {
        ok = false;
      }
    }
    if (!ok) {
      latch(R.ctl, kStRange);
      s = e = 0;
    }
    R.spans[2 * j] = s;
    R.spans[2 * j + 1] = e;
  }
}

// One workgroup of 1024 threads: exclusive prefix sums of output lengths and
// covering-block counts, in chunks of 1024 requests.
__global__ void __launch_bounds__(1024) k_req_scan(ReqArgs R) {
  __shared__ uint64_t wsum[2][16];
  const uint32_t t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const uint32_t nreq = R.ctl[kCtlNReq];
  uint64_t carry_len = 0, carry_cnt = 0;
  for (uint32_t c0 = 0; c0 < nreq; c0 += 1024) {
    const uint32_t j = c0 + t;
    uint64_t len = 0, cnt = 0;
    if (j < nreq) {
      const uint64_t s = R.spans[2 * j], e = R.spans[2 * j + 1];
      len = e - s;
      cnt = e > s ? ((e - 1) >> R.bl) - (s >> R.bl) + 1 : 0;
    }
    uint64_t il = len, ic = cnt;
    for (int d = 1; d < 64; d <<= 1) {
      const uint64_t yl = __shfl_up(il, d, 64), yc = __shfl_up(ic, d, 64);
      if (lane >= (uint32_t)d) { il += yl; ic += yc; }
    }
    if (lane == 63) { wsum[0][wv] = il; wsum[1][wv] = ic; }
    __syncthreads();
    uint64_t bl = 0, bc = 0, tl = 0, tc = 0;
    for (uint32_t q = 0; q < 16; q++) {
      if (q < wv) { bl += wsum[0][q]; bc += wsum[1][q]; }
      tl += wsum[0][q];
      tc += wsum[1][q];
    }
    if (j < nreq) {
      R.offs[j] = carry_len + bl + il - len;
      R.cnt_ptr[j] = carry_cnt + bc + ic - cnt;
      if (R.offsets) R.offsets[j] = carry_len + bl + il - len;
    }
    carry_len += tl;
    carry_cnt += tc;
    __syncthreads();
  }
  if (t == 0) {
    R.offs[nreq] = carry_len;
    R.cnt_ptr[nreq] = carry_cnt;
    if (R.offsets) R.offsets[nreq] = carry_len;
    *ctl64(R.ctl, kCtlTotal) = carry_len;
    if (carry_len > R.cap) {
      latch(R.ctl, kStCapacity);
      carry_cnt = 0;           // nothing is decoded or gathered
    }
    *ctl64(R.ctl, kCtlPairs) = carry_cnt;
  }
}

__global__ void k_req_mark(ReqArgs R) {
  const uint64_t pairs = *ctl64(R.ctl, kCtlPairs);
  const uint32_t nreq = R.ctl[kCtlNReq];
  const uint32_t epoch = R.ctl[kCtlREpoch];
  for (uint64_t g = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; g < pairs; g += (uint64_t)gridDim.x * blockDim.x) {
    const uint32_t j = find_req(R.cnt_ptr, nreq, g);
    const uint64_t b = (R.spans[2 * j] >> R.bl) + (g - R.cnt_ptr[j]);
    mark_push(R, (uint32_t)b, epoch);
  }
}

// Transitive closure over the dependency lists with a shared worklist.
// Control flow is uniform per wave (lanes of a wave cannot wait for each
// other): a wave takes 64 consecutive list indices, expands those already
// pushed (tail), and keeps the rest pending.  An expansion pushes the block's
// unmarked dependencies and then counts itself done with release order; with
// nothing ready, the wave loads done with acquire order and then tail: done ==
// tail means no entry is in flight and none can appear, so the pending indices
// stay empty and the wave stops.
__global__ void k_closure(ReqArgs R, uint32_t spin_limit) {
  const uint32_t lane = lane_id();
  const uint32_t epoch = aload(R.ctl + kCtlREpoch);
  for (;;) {
    uint32_t i0 = 0;
    if (lane == 0) i0 = __hip_atomic_fetch_add(R.ctl + kCtlListHead, 64u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    i0 = __shfl(i0, 0, 64);
    const uint32_t i = i0 + lane;
    bool pending = true;
    uint32_t spins = 0;
    while (__ballot(pending)) {
      const uint32_t tail = __shfl(aload(R.ctl + kCtlListTail), 0, 64);
      const bool ready = pending && i < tail;
      if (__ballot(ready)) {
        if (ready) {
          uint64_t v;
          uint32_t sp = 0;
          while (((v = __hip_atomic_load(R.list + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) >> 32) != epoch) {
            if (++sp > spin_limit) { watchdog(R.ctl, 2, i, (uint32_t)v, (uint32_t)(v >> 32), epoch); break; }
            __builtin_amdgcn_s_sleep(1);
          }
          const uint32_t b = (uint32_t)v;
          if ((v >> 32) == epoch) {
            const uint64_t d0 = ld64(R.arc + R.off_dep_ptr + 8ull * b), d1 = ld64(R.arc + R.off_dep_ptr + 8ull * (b + 1));
            for (uint64_t k = d0; k < d1; k++) mark_push(R, ld32(R.arc + R.off_dep_idx + 4 * k), epoch);
          }
          __hip_atomic_fetch_add(R.ctl + kCtlListDone, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
          pending = false;
        }
        spins = 0;
        continue;
      }
      const uint32_t done = __shfl(__hip_atomic_load(R.ctl + kCtlListDone, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT), 0, 64);
      const uint32_t tail2 = __shfl(aload(R.ctl + kCtlListTail), 0, 64);
      if (done == tail2 && !__ballot(pending && i < tail2)) return;   // pending indices past the end
      if (++spins > spin_limit) {
        if (lane == 0) watchdog(R.ctl, 3, i0, done, tail2, epoch);
        return;
      }
      __builtin_amdgcn_s_sleep(1);
    }
  }
}

__device__ __forceinline__ uint32_t block_level(const ReqArgs& R, uint32_t b) {
  const uint8_t* e = R.arc + R.off_dir + (uint64_t)b * kDirEntry + 20;
  return min((uint32_t)e[0] | ((uint32_t)e[1] << 8), 63u);
}

// Counters of a level are shared by every block of it: a workgroup counts in
// LDS and adds its sums once (an atomic a block was 26 us for 8192 blocks).
__global__ void __launch_bounds__(256) k_req_levels(ReqArgs R) {
  __shared__ uint32_t lvl[64];
  if (threadIdx.x < 64) lvl[threadIdx.x] = 0;
  __syncthreads();
  const uint32_t cnt = R.ctl[kCtlListTail];
  const uint64_t B = 1ull << R.bl;
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < cnt; i += gridDim.x * blockDim.x) {
    const uint32_t b = (uint32_t)R.list[i];
    atomicAdd(&lvl[block_level(R, b)], 1u);
    const uint64_t sb = (uint64_t)b << R.bl, eb = min(sb + B, R.n);
    uint64_t a = 0;
    if (R.direct && sb >= R.a0 && eb <= R.a0 + R.b0 && ((sb - R.a0) & 15) == 0) {
      a = reinterpret_cast<uint64_t>(R.out + (sb - R.a0));
    } else {
      const uint32_t slot = atomicAdd(R.ctl + kCtlSlots, 1u);
      if (slot < R.max_slots) a = reinterpret_cast<uint64_t>(R.slots + (uint64_t)slot * B);
      else latch(R.ctl, kStCapacity);
    }
    R.addr[b] = a;
  }
  __syncthreads();
  if (threadIdx.x < 64 && lvl[threadIdx.x]) atomicAdd(R.ctl + kCtlLevelCnt + threadIdx.x, lvl[threadIdx.x]);
}

__global__ void k_req_level_scan(ReqArgs R) {
  if (threadIdx.x == 0) {
    uint32_t s = 0;
    for (uint32_t L = 0; L < 64; L++) {
      R.rlevel_ptr[L] = s;
      R.rlevel_ptr[65 + L] = s;
      s += R.ctl[kCtlLevelCnt + L];
    }
    R.rlevel_ptr[64] = s;
  }
}

__global__ void __launch_bounds__(256) k_req_scatter(ReqArgs R) {
  __shared__ uint32_t lvl[64];
  const uint32_t t = threadIdx.x, cnt = R.ctl[kCtlListTail];
  for (uint32_t i0 = blockIdx.x * 256; i0 < cnt; i0 += gridDim.x * 256) {       // uniform
    if (t < 64) lvl[t] = 0;
    __syncthreads();
    const bool have = i0 + t < cnt;
    const uint32_t b = have ? (uint32_t)R.list[i0 + t] : 0u, L = have ? block_level(R, b) : 0u;
    const uint32_t k = have ? atomicAdd(&lvl[L], 1u) : 0u;
    __syncthreads();
    if (t < 64 && lvl[t]) lvl[t] = atomicAdd(R.rlevel_ptr + 65 + t, lvl[t]);    // the level's next places
    __syncthreads();
    if (have) R.rqueue[lvl[L] + k] = b;
    __syncthreads();
  }
}

// Plan of a small request call in one workgroup of 1024 threads, the same
// steps as k_req_begin .. k_req_scatter without launches between them: clear
// the previous closure's addresses, spans and prefix sums of the requests,
// covering blocks marked and listed, the dependency closure expanded round by
// round (a round takes every listed entry not yet expanded; a block joins the
// list once, when it is marked), then a counting sort of the closure by level
// with each block's address.  Bound by the latency of each step, so marks,
// list and levels are kept in LDS as far as they fit: marks as bits of at
// most kPlanBits blocks (R.lmark; else as epochs in memory), the first
// kPlanList entries of list and levels.  4096 records on 8192 blocks: 175 us
// for the eight kernels, 55 us here; 256 mixed requests 86 and 19 us.
constexpr uint32_t kPlanWG = 1024;
constexpr uint32_t kPlanBits = 1u << 18, kPlanList = 6144;
constexpr uint32_t kPlanOwn = 8;       // covering blocks that a request's own thread marks

__global__ void __launch_bounds__(kPlanWG) k_req_plan(ReqArgs R) {
  __shared__ uint32_t s_bits[kPlanBits / 32], s_list[kPlanList];
  __shared__ uint8_t s_lvl[kPlanList];
  __shared__ uint64_t wsum[2][kPlanWG / 64];
  __shared__ uint32_t lvl_cnt[64], lvl_cur[64];
  __shared__ uint32_t s_tail, s_slots, s_nreq, s_epoch;
  __shared__ uint64_t s_pairs;
  const uint32_t t = threadIdx.x, lane = t & 63, wv = t >> 6;
  // begin: the previous call's closure loses its addresses; new epochs
  {
    const uint32_t prev = min(R.ctl[kCtlListTail], (uint32_t)R.n_blocks);
    for (uint32_t i = t; i < prev; i += kPlanWG) {
      const uint32_t b = (uint32_t)R.list[i];
      if (b < R.n_blocks) R.addr[b] = 0;
    }
  }
  const bool renew = renew_flags(R);
  if (R.lmark)
    for (uint32_t i = t; i < ((uint32_t)R.n_blocks + 31) / 32; i += kPlanWG) s_bits[i] = 0;
  if (t < 64) lvl_cnt[t] = 0;
  if (t == 0) {
    uint64_t n = R.n_max;
    if (R.mode == 2) n = min((uint64_t)*R.d_n, R.n_max);
    s_nreq = (uint32_t)n;
    s_tail = 0;
    s_slots = 0;
    s_epoch = R.ctl[kCtlREpoch] + 1;
    R.ctl[kCtlREpoch] = s_epoch;
    R.ctl[kCtlListHead] = 0;
    R.ctl[kCtlListDone] = 0;
    R.ctl[kCtlNReq] = (uint32_t)n;
  }
  __syncthreads();
  const uint32_t epoch = s_epoch;
  const uint32_t nreq = s_nreq;
  if (renew && t == 0) R.ctl[kCtlEpoch] = 0;
  // spans, output offsets and covering-block counts, 1024 requests a round
  uint64_t carry_len = 0, carry_cnt = 0;
  for (uint32_t c0 = 0; c0 < nreq; c0 += kPlanWG) {
    const uint32_t j = c0 + t;
    uint64_t s0 = 0, e0 = 0;
    if (j < nreq) {
      bool ok = true;
      if (R.mode == 0) {
        s0 = R.a0;
        e0 = R.a0 + R.b0;
      } else if (R.mode == 1) {
        ok = read_span(R, R.ids[j], s0, e0);
      } else {
        const lz_request q = R.reqs[j];
        if (q.kind == 0) {
          ok = read_span(R, q.a, s0, e0);
        } else if (q.kind == 1 && q.a >= 0 && q.b >= 0 && (uint64_t)q.a <= R.n && (uint64_t)q.b <= R.n - (uint64_t)q.a) {
          s0 = (uint64_t)q.a;
          e0 = s0 + (uint64_t)q.b;
        } else {
          ok = false;
        }
      }
      if (!ok) {
        latch(R.ctl, kStRange);
        s0 = e0 = 0;
      }
      R.spans[2 * j] = s0;
      R.spans[2 * j + 1] = e0;
    }
    const uint64_t len = e0 - s0;
    const uint64_t cnt = e0 > s0 ? ((e0 - 1) >> R.bl) - (s0 >> R.bl) + 1 : 0;
    uint64_t il = len, ic = cnt;
    for (int d = 1; d < 64; d <<= 1) {
      const uint64_t yl = __shfl_up(il, d, 64), yc = __shfl_up(ic, d, 64);
      if (lane >= (uint32_t)d) { il += yl; ic += yc; }
    }
    if (lane == 63) { wsum[0][wv] = il; wsum[1][wv] = ic; }
    __syncthreads();
    uint64_t bl = 0, bc = 0, tl = 0, tc = 0;
    for (uint32_t q = 0; q < kPlanWG / 64; q++) {
      if (q < wv) { bl += wsum[0][q]; bc += wsum[1][q]; }
      tl += wsum[0][q];
      tc += wsum[1][q];
    }
    if (j < nreq) {
      R.offs[j] = carry_len + bl + il - len;
      R.cnt_ptr[j] = carry_cnt + bc + ic - cnt;
      if (R.offsets) R.offsets[j] = carry_len + bl + il - len;
    }
    carry_len += tl;
    carry_cnt += tc;
    __syncthreads();
  }
  if (t == 0) {
    R.offs[nreq] = carry_len;
    R.cnt_ptr[nreq] = carry_cnt;
    if (R.offsets) R.offsets[nreq] = carry_len;
    *ctl64(R.ctl, kCtlTotal) = carry_len;
    uint64_t pairs = carry_cnt;
    if (carry_len > R.cap) {
      latch(R.ctl, kStCapacity);
      pairs = 0;                 // nothing is decoded or gathered
    }
    *ctl64(R.ctl, kCtlPairs) = pairs;
    s_pairs = pairs;
  }
  __syncthreads();
  // covering blocks: marked and listed once each
  const uint64_t pairs = s_pairs;
  auto push = [&](uint32_t b) {
    if (R.lmark) {
      if (b >= R.n_blocks || (atomicOr(&s_bits[b >> 5], 1u << (b & 31)) >> (b & 31)) & 1u) return;
    } else {
      const uint32_t old = __hip_atomic_fetch_max(R.mark + b, epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (old >= epoch) return;
    }
    const uint32_t i = atomicAdd(&s_tail, 1u);
    if (i < kPlanList) s_list[i] = b;
    if (i < R.n_blocks) R.list[i] = ((uint64_t)epoch << 32) | b;
  };
  auto listed = [&](uint32_t i) { return i < kPlanList ? s_list[i] : (uint32_t)R.list[i]; };
  if (R.mode == 0) {
    for (uint64_t g = t; g < pairs; g += kPlanWG) push((uint32_t)((R.a0 >> R.bl) + g));
  } else if (pairs) {
    // a thread per request for its first blocks, then the wave together for
    // each request that has more, one such request after the other: with its
    // share at 4, 100 records of six blocks of 64 bytes each took that turn
    // (18 us of a call of 86; from 16 on a lone thread holds the others up)
    for (uint32_t c0 = 0; c0 < nreq; c0 += kPlanWG) {
      const uint32_t j = c0 + t;
      uint32_t b0 = 0, n = 0;
      if (j < nreq) {
        const uint64_t s0 = R.spans[2 * j], e0 = R.spans[2 * j + 1];
        b0 = (uint32_t)(s0 >> R.bl);
        n = e0 > s0 ? (uint32_t)(((e0 - 1) >> R.bl) - b0 + 1) : 0u;
      }
      for (uint32_t k = 0; k < min(n, kPlanOwn); k++) push(b0 + k);
      for (uint64_t more = __ballot(n > kPlanOwn); more; more &= more - 1) {     // wave-uniform
        const uint32_t l = (uint32_t)__builtin_ctzll(more);
        const uint32_t nb = __builtin_amdgcn_readlane(n, l), bb = __builtin_amdgcn_readlane(b0, l);
        for (uint32_t k = kPlanOwn + lane; k < nb; k += 64) push(bb + k);
      }
    }
  }
  __syncthreads();
  // dependency closure, one round per pass over the entries listed so far.
  // Every thread reads the round's tail between two barriers, before anyone
  // pushes in this round: a wave reading it after another wave's pushes would
  // see a longer list, and threads leaving the loop in different rounds would
  // meet at different barriers.
  uint32_t head = 0;
  for (uint32_t round = 0; round <= R.n_blocks; round++) {
    const uint32_t tail = min(s_tail, (uint32_t)R.n_blocks);
    __syncthreads();
    if (head >= tail) break;
    for (uint32_t i = head + t; i < tail; i += kPlanWG) {
      const uint32_t b = listed(i);
      const uint64_t d0 = ld64(R.arc + R.off_dep_ptr + 8ull * b), d1 = ld64(R.arc + R.off_dep_ptr + 8ull * (b + 1));
      for (uint64_t k = d0; k < d1; k += 4) {
        uint32_t id[4];
#pragma unroll
        for (uint32_t u = 0; u < 4; u++) id[u] = k + u < d1 ? ld32(R.arc + R.off_dep_idx + 4 * (k + u)) : 0u;
#pragma unroll
        for (uint32_t u = 0; u < 4; u++)
          if (k + u < d1) push(id[u]);
      }
    }
    head = tail;
    __syncthreads();
  }
  const uint32_t cnt = min(s_tail, (uint32_t)R.n_blocks);
  // levels and addresses: straight into the output for a block wholly inside
  // an aligned single range, else a scratch slot
  const uint64_t B = 1ull << R.bl;
  for (uint32_t i = t; i < cnt; i += kPlanWG) {
    const uint32_t b = listed(i), L = block_level(R, b);
    if (i < kPlanList) s_lvl[i] = (uint8_t)L;
    atomicAdd(&lvl_cnt[L], 1u);
    const uint64_t sb = (uint64_t)b << R.bl, eb = min(sb + B, R.n);
    uint64_t a = 0;
    if (R.direct && sb >= R.a0 && eb <= R.a0 + R.b0 && ((sb - R.a0) & 15) == 0) {
      a = reinterpret_cast<uint64_t>(R.out + (sb - R.a0));
    } else {
      const uint32_t slot = atomicAdd(&s_slots, 1u);
      if (slot < R.max_slots) a = reinterpret_cast<uint64_t>(R.slots + (uint64_t)slot * B);
      else latch(R.ctl, kStCapacity);
    }
    R.addr[b] = a;
  }
  __syncthreads();
  if (t < 64) {                                 // exclusive scan of the 64 level counts
    const uint32_t c = lvl_cnt[t];
    uint32_t incl = c;
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t y = __shfl_up(incl, d, 64);
      if (t >= (uint32_t)d) incl += y;
    }
    R.rlevel_ptr[t] = incl - c;
    R.rlevel_ptr[65 + t] = incl - c;
    lvl_cur[t] = incl - c;
    if (t == 63) R.rlevel_ptr[64] = incl;
  }
  __syncthreads();
  for (uint32_t i = t; i < cnt; i += kPlanWG) {
    const uint32_t b = listed(i);
    R.rqueue[atomicAdd(&lvl_cur[i < kPlanList ? s_lvl[i] : block_level(R, b)], 1u)] = b;
  }
  if (t == 0) {
    R.ctl[kCtlListTail] = cnt;
    R.ctl[kCtlSlots] = s_slots;
    if (s_tail > R.n_blocks) latch(R.ctl, kStCorrupt);
  }
}

// The same as find_req with every lane of a wave probing: 64 probes a step,
// so two dependent loads for 4096 requests instead of twelve.
__device__ __forceinline__ uint32_t find_req_wave(const uint64_t* v, uint32_t n, uint64_t g) {
  const uint32_t lane = lane_id();
  uint32_t lo = 0, len = n;
  while (len > 1) {
    const uint32_t step = (len + 63) >> 6, at = lane * step;
    const uint64_t le = __ballot(at < len && v[lo + min(at, len - 1)] <= g);   // a prefix: v is sorted
    const uint32_t k = (uint32_t)__popcll(le) - 1;                             // v[lo] <= g
    lo += k * step;
    len = min(step, len - k * step);
  }
  return lo;
}

// n bytes from src to dst by one wave, any alignment: 16-byte stores aligned
// in dst (the loads need no alignment), up to 15 bytes at each end one by one.
// All loads of a 4 KiB round go out before its stores.
__device__ __forceinline__ void wave_copy(uint8_t* dst, const uint8_t* src, uint32_t n) {
  const uint32_t lane = lane_id();
  const uint32_t head = min(n, (uint32_t)(-(uintptr_t)dst & 15u));
  const uint32_t n16 = (n - head) >> 4, t0 = head + 16 * n16;
  const bool hb = lane < head, tb = t0 + lane < n;
  const uint8_t h = hb ? src[lane] : (uint8_t)0, t = tb ? src[t0 + lane] : (uint8_t)0;
  u32x4* d4 = reinterpret_cast<u32x4*>(dst + head);
  for (uint32_t c = 0; c < n16; c += 256) {
    u32x4 v[4] = {};
#pragma unroll
    for (uint32_t u = 0; u < 4; u++) {
      const uint32_t i = c + 64 * u + lane;
      if (i < n16) v[u] = ld128(src + head + 16 * (uint64_t)i);
    }
#pragma unroll
    for (uint32_t u = 0; u < 4; u++) {
      const uint32_t i = c + 64 * u + lane;
      if (i < n16) d4[i] = v[u];
    }
  }
  if (hb) dst[lane] = h;
  if (tb) dst[t0 + lane] = t;
}

// Requested parts of blocks that were decoded into scratch slots, copied to
// the output: one wave per part of a (request, covering block) pair, `parts`
// parts to a block.  Bound by memory, so what counts is enough bytes in
// flight: a grid sized by the bytes asked for (one workgroup per 256 blocks of
// the file, a byte a thread, was 1506 us for 48 MiB of misaligned range).
__global__ void __launch_bounds__(256) k_req_gather(ReqArgs R, uint32_t parts) {
  const uint64_t pairs = *ctl64(R.ctl, kCtlPairs);
  const uint32_t nreq = R.ctl[kCtlNReq];
  const uint64_t B = 1ull << R.bl, P = B / parts, waves = (uint64_t)gridDim.x * 4;
  for (uint64_t w = (uint64_t)blockIdx.x * 4 + uni(threadIdx.x >> 6); w < pairs * parts; w += waves) {
    const uint64_t g = w / parts;
    const uint32_t j = find_req_wave(R.cnt_ptr, nreq, g);
    const uint64_t s = R.spans[2 * j], e = R.spans[2 * j + 1];
    const uint64_t b = (s >> R.bl) + (g - R.cnt_ptr[j]);
    const uint64_t a = R.addr[b];
    if (!a) continue;
    const uint64_t sb = b << R.bl, p0 = sb + (w - g * parts) * P;
    const uint64_t lo = max(p0, s), hi = min(min(p0 + P, R.n), e);
    if (hi <= lo) continue;
    uint8_t* dst = R.out + R.offs[j] + (lo - s);
    const uint8_t* src = reinterpret_cast<const uint8_t*>(a) + (lo - sb);
    if (src == dst) continue;   // decoded in place
    wave_copy(dst, src, (uint32_t)(hi - lo));
  }
}

// The same by one workgroup, a byte a thread (see lz_launch_requests).
__global__ void __launch_bounds__(256) k_req_gather_one(ReqArgs R) {
  const uint64_t pairs = *ctl64(R.ctl, kCtlPairs);
  const uint32_t nreq = R.ctl[kCtlNReq];
  const uint64_t B = 1ull << R.bl;
  for (uint64_t g = 0; g < pairs; g++) {
    const uint32_t j = find_req(R.cnt_ptr, nreq, g);
    const uint64_t s = R.spans[2 * j], e = R.spans[2 * j + 1];
    const uint64_t b = (s >> R.bl) + (g - R.cnt_ptr[j]);
    const uint64_t a = R.addr[b];
    if (!a) continue;
    const uint64_t sb = b << R.bl, lo = max(sb, s), hi = min(min(sb + B, R.n), e);
    if (hi <= lo) continue;
    uint8_t* dst = R.out + R.offs[j] + (lo - s);
    const uint8_t* src = reinterpret_cast<const uint8_t*>(a) + (lo - sb);
    for (uint64_t q = threadIdx.x; q < hi - lo; q += blockDim.x) dst[q] = src[q];
  }
}

}  // namespace

int lz_launch_requests(lz_handle* h, const lz_request* d_reqs, const uint32_t* d_n, uint64_t n_max,
                       uint64_t single_off, uint64_t single_len, const int64_t* d_ids,
                       uint8_t* d_out, uint64_t cap, uint64_t* d_offsets, void* d_scratch,
                       uint64_t scratch_len, hipStream_t s) {
  const ArchiveView& v = h->av;
  ReqArgs R{};
  R.arc = v.base;
  R.n = v.n;
  R.n_blocks = v.n_blocks;
  R.off_dir = v.off_dir;
  R.off_dep_ptr = v.off_dep_ptr;
  R.off_dep_idx = v.off_dep_idx;
  R.off_ridx = v.kind == 1 ? v.off_ridx : 0;
  R.n_reads = v.n_reads;
  R.bl = v.block_log2;
  R.mode = d_reqs ? 2u : (d_ids ? 1u : 0u);
  R.a0 = single_off;
  R.b0 = single_len;
  R.ids = d_ids;
  R.reqs = d_reqs;
  R.d_n = d_n;
  R.n_max = n_max;
  R.out = d_out;
  R.cap = cap;
  R.offsets = d_offsets;
  // scratch: spans, block-count prefix, output prefix, then 16 KiB slots
  const uint64_t B = 1ull << v.block_log2;
  uint8_t* sc = reinterpret_cast<uint8_t*>(d_scratch);
  if (!sc || ((uintptr_t)sc & 255)) return lz_fail(LZ_EINVAL, "request scratch must be 256-byte aligned");
  const uint64_t spans_b = 16 * n_max, ptr_b = 8 * (n_max + 1);
  const uint64_t slots_off = (spans_b + 2 * ptr_b + 255) & ~255ull;
  if (scratch_len < slots_off) return lz_fail(LZ_ECAPACITY, "request scratch needs at least %llu bytes", (unsigned long long)slots_off);
  R.spans = reinterpret_cast<uint64_t*>(sc);
  R.cnt_ptr = reinterpret_cast<uint64_t*>(sc + spans_b);
  R.offs = reinterpret_cast<uint64_t*>(sc + spans_b + ptr_b);
  R.slots = sc + slots_off;
  R.max_slots = (scratch_len - slots_off) / B;
  R.direct = (R.mode == 0 && ((uintptr_t)d_out & 15) == 0) ? 1u : 0u;
  R.mark = h->ws.mark;
  R.flags = h->ws.flags;
  R.addr = h->ws.addr;
  R.rqueue = h->ws.rqueue;
  R.rlevel_ptr = h->ws.rlevel_ptr;
  R.list = h->ws.list;
  R.ctl = h->ws.ctl;
  const uint32_t spin = h->tune.spin_limit ? h->tune.spin_limit : (1u << 20);
  const uint32_t g_req = (uint32_t)std::min<uint64_t>(1024, (n_max + 255) / 256);
  // small calls are planned by one workgroup (one launch instead of eight):
  // at most plan_blocks covering blocks expected (a range; a record lies in one
  // block or a few more; of a batch 256 blocks a request, but not more than
  // its output holds)
  const uint64_t Bs = 1ull << v.block_log2, pb = h->tune.plan_blocks ? h->tune.plan_blocks : 4096;
  const uint64_t covering = R.mode == 0 ? single_len / Bs + 2
                          : R.mode == 1 ? n_max * (v.max_record_len / Bs + 1)
                                        : std::min(n_max * 256, cap / Bs + 2 * n_max);
  const bool small = pb > 1 && covering <= pb;     // 1: never
  R.lmark = v.n_blocks <= kPlanBits ? 1u : 0u;
  const uint32_t g_wide = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(1024, (v.n_blocks + 255) / 256));
  if (small) {
    hipLaunchKernelGGL(k_req_plan, dim3(1), dim3(kPlanWG), 0, s, R);
  } else {
    hipLaunchKernelGGL(k_req_begin, dim3(1), dim3(256), 0, s, R);
    hipLaunchKernelGGL(k_req_spans, dim3(g_req), dim3(256), 0, s, R);
    hipLaunchKernelGGL(k_req_scan, dim3(1), dim3(1024), 0, s, R);
    hipLaunchKernelGGL(k_req_mark, dim3(g_wide), dim3(256), 0, s, R);
    hipLaunchKernelGGL(k_closure, dim3(std::min<uint32_t>(64, g_wide)), dim3(256), 0, s, R, spin);
    hipLaunchKernelGGL(k_req_levels, dim3(g_wide), dim3(256), 0, s, R);
    hipLaunchKernelGGL(k_req_level_scan, dim3(1), dim3(64), 0, s, R);
    hipLaunchKernelGGL(k_req_scatter, dim3(g_wide), dim3(256), 0, s, R);
  }
  // decode the closure in level order (one launch, or one per level)
  DevArgs A = make_args(h);
  A.queue = h->ws.rqueue;
  A.qptr = h->ws.rlevel_ptr;
  A.addr = h->ws.addr;
  A.out = d_out;
  const uint32_t grid = (uint32_t)std::min<uint64_t>(decode_slots(h), std::max<uint64_t>(1, v.n_blocks));
  // the closure, which is known on the device only, taken as three times the
  // covering blocks; of a small archive half the blocks at most
  const bool levels = shallow(h, std::min(3 * std::min(covering, v.n_blocks), v.n_blocks / 2));
  if (h->tune.req_sync_mode == 0 && h->deps_listed && v.n_levels > 1 && !levels) {
    // scratch slots are whole lines; blocks decoded straight into the output lie
    // at d_out - single_off plus a multiple of the block size
    const uint64_t at = reinterpret_cast<uintptr_t>(d_out) - single_off;
    A.flow = flow_mode(A, R.direct && (at & 15) == 0 ? at : 0);
    A.q_end = kMaxLevels;                  // rlevel_ptr[0] .. rlevel_ptr[64]: the whole closure
    launch_decode(A, grid, s);
  } else {
    for (uint32_t L = 0; L < v.n_levels; L++) {
      A.q_begin = L;
      A.q_end = L + 1;
      launch_decode(A, grid, s);
    }
  }
  // gather: a wave copies up to a quarter of a block (4 KiB in flight); records
  // are short, so a wave takes what a record has in a block
  const uint32_t parts = R.mode == 1 || Bs < 256 ? 1u : 4u;
  const uint64_t pairs = R.mode == 0 ? single_len / Bs + 2
                       : R.mode == 1 ? n_max * (v.max_record_len / Bs + 2)
                                     : std::min<uint64_t>(cap / Bs, v.n_blocks * n_max) + 2 * n_max;
  const uint64_t g_gather = (pairs * parts + 3) / 4;
  // Batches on an archive of less than 256 blocks stay with one workgroup: a
  // program that serves such an archive (tests/test_gpu_serve.py) counts on a
  // batch of 3 MiB being on the device for the millisecond in which the next
  // ones arrive (3 ms so, 0.14 ms with the grid below).  The streams of a split
  // container are not served so: 266 reads of a 1.3 MB one 1640 us with one
  // workgroup a stream, 195 us with the grid.
  if (R.mode == 2 && v.n_blocks < 256 && !h->of_split)
    hipLaunchKernelGGL(k_req_gather_one, dim3(1), dim3(256), 0, s, R);
  else
    hipLaunchKernelGGL(k_req_gather, dim3((uint32_t)std::min<uint64_t>(g_gather, 16ull * h->n_cu)), dim3(256), 0, s, R, parts);
  return launch_ok("request decode");
}
