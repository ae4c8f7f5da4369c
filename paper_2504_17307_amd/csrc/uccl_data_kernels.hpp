// Data-path kernels: dedup of a tile of records, the kernel that streams the winners (whole tiles
// per workgroup, or one record cut into parts over several workgroups), the multi-source fold,
// and the bitmap fill.  Internal to the library: included by uccl_chunk.hip only.
#pragma once

#include "uccl_chunk.h"
#include "uccl_elements.hpp"

// Tunable compile-time shape constants (defaults chosen by measurement on MI355X).
#ifndef UCCL_GATHER_UNROLL
#define UCCL_GATHER_UNROLL 2  // multi-sender reduce: vectors per lane per unit
#endif
#ifndef UCCL_GATHER_BATCH
#define UCCL_GATHER_BATCH 4   // and how many sources are loaded before the folds start
#endif
#ifndef UCCL_FLAT_THREADS
#define UCCL_FLAT_THREADS 1024  // workgroup size of chunk_flat_kernel
#endif
#ifndef UCCL_FLAT_UNROLL
#define UCCL_FLAT_UNROLL 2    // vectors per lane per unit: a unit is 64*U*16 bytes per stream
#endif
#ifndef UCCL_FLAT1_REDUCE_UNROLL
#define UCCL_FLAT1_REDUCE_UNROLL 1  // the same for one-record tiles of kernels that read the accumulator
#endif
#ifndef UCCL_FEW_THREADS
#define UCCL_FEW_THREADS 1024   // calls of few records: one workgroup per record
#endif
#ifndef UCCL_FEW_UNROLL
#define UCCL_FEW_UNROLL 4
#endif
#ifndef UCCL_PART_THREADS
#define UCCL_PART_THREADS 256   // workgroup size when one record is cut into parts
#endif
#ifndef UCCL_PART_UNROLL
#define UCCL_PART_UNROLL 2
#endif
#ifndef UCCL_XCD_CONTIGUOUS
#define UCCL_XCD_CONTIGUOUS 0   // 1: chunk_flat_kernel gives each of the 8 XCDs one contiguous eighth of the tiles
#endif
#ifndef UCCL_CLAIM_STRIDE
#define UCCL_CLAIM_STRIDE 16    // 64-bit words from one record's claim word to the next: one 128-byte line each
#endif
#ifndef UCCL_CLAIM_SPIN_LIMIT
#define UCCL_CLAIM_SPIN_LIMIT (1u << 16)  // polls of a claim word before a part gives up (see claim_await)
#endif
// At most 80 scalar and 64 vector registers a wavefront: eight wavefronts on a SIMD (with 86 scalar ones the hardware
// holds seven).
#define UCCL_FULL_OCCUPANCY __attribute__((amdgpu_num_sgpr(80), amdgpu_waves_per_eu(8)))
namespace {

struct Extents {
  uint64_t acc_bytes, out_bytes, recv_bytes, n_bits;
};

// What the claim words of a call (see claim_enter) are: its share of them, its own tag, workgroups per record, and
// where, from `claims`, the 64-bit word lies that counts the parts that gave up waiting.
//
// 112 bytes of arguments are what HIP launches at full speed; from 120 on a launch takes the host 0.65 us more (2.70 / 3.35
// us in a loop of launches, 0.05 in a process in which launches are faster): so the words are packed.
struct ClaimArgs {
  unsigned long long* claims;
  uint32_t parts : 16;
  unsigned long long tag : 48;
  uint32_t faults_at : 31;
  uint32_t allow_forward : 1;
  uint32_t n_descs;

  __host__ __device__ uint32_t* faults() const { return reinterpret_cast<uint32_t*>(claims + faults_at); }
  void use(unsigned long long* words, const void* counter) {
    claims = words;
    faults_at = static_cast<uint32_t>(static_cast<const unsigned long long*>(counter) - words);
  }
};
static_assert(sizeof(ClaimArgs) == 24, "packed");

template <class Desc>
struct Buffers {
  char* acc;
  char* out;
  const char* recv;
  const Desc* descs;
  uint32_t* bitmap;
  uint32_t* rejected;
  Extents ext;
};

struct Args : Buffers<uccl_chunk_desc>, ClaimArgs {
  const uint32_t* n_ptr;  // optional: the record count is read from here (capped by n_descs)
};
static_assert(sizeof(Args) == 112, "see ClaimArgs");

// ---- one record, several workgroups ------------------------------------------------------
//
// A call of few, large records (a 4 MiB message in 64 KiB chunks is 57 of them per phase) puts
// one workgroup per record on the machine, and a single compute unit moves its 4 x 64 KiB far
// below its share of the memory system's rate.  Such a call is launched with `parts` workgroups
// per record, and the record's units are dealt over the wavefronts of all of them.  The sequence
// number must still be decided exactly once, by one atomic OR on the bitmap, and every part that
// has units must learn the outcome.  Record k of the call has a 64-bit claim word in scratch
// memory, holding `tag << 16 | state`: the tag of the last call that used the word, and 0 = a part
// is deciding, 1 = applied, 2 = not applied.  No two calls have the same tag.
//
//   enter    every part issues one atomic max of `tag << 16` on the word, after the payload loads of
//            its first unit (memory operations return in order, so entering earlier would hold up
//            the record itself).  Tags grow from call to call in the order the calls run (the host
//            draws the tag and enqueues the launch under one lock, and calls that share a word run
//            on one stream), so exactly one part of the call -- the first to get there -- finds an
//            older tag in the word: it decides.
//   decide   the deciding part issues the bitmap atomic (or rejects the record) and stores
//            `tag << 16 | outcome`.  It waits for nothing.
//   await    the other parts poll the word until it carries the call's tag and an outcome.
//
// The no-allocation calls share their words over all streams, so the order in which calls run need not be that of
// their tags.  There (APART) a part exchanges the word instead and decides if it finds any other tag, and the
// outcome is in the next word, where no part that comes later can overwrite it.  Every part then waits for one
// more load, which costs a call of many parts more (fold of 65 x 128 KiB from three senders, 16 parts, 9.4 -> 10.6 us;
// 28 records in 8 parts nothing that can be measured), so calls with a region of their own have the other way, in
// a kernel of its own (choosing at run time costs a 4 MiB ring step 2 %).
//
// A part only ever waits for a part that is already running and never waits itself, so the wait
// ends whatever order the hardware starts workgroups in.  It is bounded all the same: a part that
// gives up counts itself in `faults` and streams nothing.  Claim words are read and written with
// device-scope atomics only, so every part sees the one coherent copy whichever XCD it runs on;
// each record's word has a 128-byte line to itself (UCCL_CLAIM_STRIDE), because device-scope atomics
// on one line are served one after the other and a call's parts all arrive at about the same time
// (57 records x 8 parts: 6.2 us per call with the words packed, 5.4 us with a line each).
// Nothing is ever cleared between calls: a stale word is recognised by its tag.  The order table
// of large calls (below) lives in the same words and carries its tag in the same bits, so either kind
// of call finds the other's leftovers stale.
struct Claim {
  bool decides;
  unsigned long long seen;   // what the word with the outcome held: the outcome may already be in it
};

template <bool APART>
__device__ __forceinline__ Claim claim_enter(unsigned long long* claim, unsigned long long tag) {
  if constexpr (!APART) {
    const unsigned long long was = __hip_atomic_fetch_max(claim, tag << 16, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return {(was >> 16) < tag, was};
  } else {
    const unsigned long long was = __hip_atomic_exchange(claim, tag << 16, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return {(was >> 16) != tag, __hip_atomic_load(claim + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)};
  }
}

template <bool APART>
__device__ __forceinline__ void claim_publish(unsigned long long* claim, unsigned long long tag, bool win) {
  __hip_atomic_store(claim + (APART ? 1 : 0), (tag << 16) | (win ? 1ull : 2ull), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <bool APART>
__device__ __forceinline__ bool claim_await(unsigned long long* claim, unsigned long long seen, unsigned long long tag, uint32_t* faults) {
  for (uint32_t polls = 0; (seen >> 16) != tag || (seen & 3ull) == 0ull; ++polls) {
    if (polls >= UCCL_CLAIM_SPIN_LIMIT) {
      atomicAdd(faults, 1u);
      return false;
    }
    __builtin_amdgcn_s_sleep(1);
    seen = __hip_atomic_load(claim + (APART ? 1 : 0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  return (seen & 3ull) == 1ull;
}

// The last len % 16 bytes of a chunk, element by element.
template <class Op, bool FWD, bool WB>
__device__ __forceinline__ void stream_tail(const char* r, char* a, char* o, uint32_t rem,
                                            uint32_t lane) {
  if constexpr (Op::kEs == 4) {
    if (lane < rem / 4) {
      uint32_t* ap = reinterpret_cast<uint32_t*>(a) + lane;
      const uint32_t t = Op::word(*ap, reinterpret_cast<const uint32_t*>(r)[lane]);
      if (WB) *ap = t;
      if (FWD) reinterpret_cast<uint32_t*>(o)[lane] = t;
    }
  } else if constexpr (Op::kEs == 2) {
    if (lane < rem / 2) {
      uint16_t* ap = reinterpret_cast<uint16_t*>(a) + lane;
      const uint32_t t = Op::half(*ap, reinterpret_cast<const uint16_t*>(r)[lane]);
      if (WB) *ap = static_cast<uint16_t>(t);
      if (FWD) reinterpret_cast<uint16_t*>(o)[lane] = static_cast<uint16_t>(t);
    }
  } else {
    if (lane < rem) {
      const char t = r[lane];
      if (WB) a[lane] = t;
      if (FWD) o[lane] = t;
    }
  }
}

// What a record must satisfy before its bit is touched (the unchecked entry points pass
// unbounded extents, which leaves alignment, granularity and the forward rules).
template <uint32_t kEs>
__device__ __forceinline__ bool record_ok(const Args& g, uint64_t src, uint64_t dst, uint64_t out,
                                          uint32_t len, uint32_t seq) {
  const bool fwd = out != UCCL_NO_FORWARD;
  const uint64_t out_at = out & ~UCCL_FORWARD_ONLY;
  bool ok = seq < g.ext.n_bits && ((src | dst) & 15u) == 0 && len % kEs == 0 &&
            src <= g.ext.recv_bytes && len <= g.ext.recv_bytes - src &&
            dst <= g.ext.acc_bytes && len <= g.ext.acc_bytes - dst;
  if (fwd)
    ok = ok && g.allow_forward && g.out != nullptr && (out_at & 15u) == 0 &&
         out_at <= g.ext.out_bytes && len <= g.ext.out_bytes - out_at;
  return ok;
}

// Winners of one tile of records, compacted; first[] is the exclusive prefix sum of
// their unit counts with the total in first[count].
template <int T>
struct Tile {
  uint64_t src[T], dst[T], out[T];
  uint32_t len[T];
  uint32_t first[T + 1];
  uint32_t count;
};

// Run by the first wavefront of a workgroup: lane i takes record tile*T + i, validates
// it, claims its sequence number, and the winners are compacted into LDS in record order.
// kUnitVecs > 0 also computes how many units of kUnitVecs 16-byte vectors each winner has.
template <int T, class Op, uint32_t kUnitVecs>
__device__ __forceinline__ void dedup_tile(const Args& g, Tile<T>& s, uint32_t tile, uint32_t tid) {
  static_assert(T >= 1 && T <= 64, "one wavefront dedups the tile");
  const uint64_t k = static_cast<uint64_t>(tile) * T + tid;
  bool win = false;
  uint64_t src = 0, dst = 0, out = 0;
  uint32_t len = 0;
  if (tid < T && k < g.n_descs) {  // inside the array's capacity: safe to load
    const u32x4* p = reinterpret_cast<const u32x4*>(g.descs + k);
    const u32x4 lo = p[0], hi = p[1];
    const uint32_t live = g.n_ptr != nullptr ? *g.n_ptr : g.n_descs;
    src = lo.x | (static_cast<uint64_t>(lo.y) << 32);
    dst = lo.z | (static_cast<uint64_t>(lo.w) << 32);
    out = hi.x | (static_cast<uint64_t>(hi.y) << 32);
    len = hi.z;
    const uint32_t seq = hi.w;
    const bool ok = record_ok<Op::kEs>(g, src, dst, out, len, seq);
    if (k >= live) {
      // beyond the published count: not a record at all, neither applied nor rejected
    } else if (ok) {
      const uint32_t bit = 1u << (seq & 31u);
      const uint32_t old = atomicOr(g.bitmap + (seq >> 5), bit);  // device scope, relaxed
      win = (old & bit) == 0;
    } else if (g.rejected != nullptr) {
      atomicAdd(g.rejected, 1u);
    }
  }
  const uint64_t winners = __ballot(win);
  const uint32_t pos = __popcll(winners & ((1ull << tid) - 1ull));
  const uint32_t count = __popcll(winners);
  if (win) {
    s.src[pos] = src;
    s.dst[pos] = dst;
    s.out[pos] = out;
    s.len[pos] = len;
  }
  if (tid == 0) s.count = count;
  if (kUnitVecs > 0) {
    // a partial last vector (len % 16 != 0) counts as a vector of its unit
    const uint32_t vecs = (len >> 4) + ((len & 15u) != 0u ? 1u : 0u);  // no overflow for len up to 2^32 - 1
    const uint32_t units = win ? (vecs + kUnitVecs - 1u) / kUnitVecs : 0u;
    uint32_t incl = units;
#pragma unroll
    for (uint32_t d = 1; d < 64; d <<= 1) {
      const uint32_t below = __shfl_up(incl, d, 64);
      if (tid >= d) incl += below;
    }
    if (win) s.first[pos] = incl - units;
    if (tid == 63) s.first[count] = incl;
  }
}

// One unit = 64*U consecutive 16-byte vectors of a chunk, streamed by one wavefront.
template <int U, class Op, bool FWD, bool WB, Through T>
__device__ __forceinline__ void stream_unit(const char* r, char* a, char* o, uint32_t len,
                                            uint32_t trip, uint32_t lane) {
  constexpr uint32_t kPolicy = cache_policy<Op, FWD, WB>();
  constexpr bool kNtRecv = (kPolicy & 8u) != 0, kNtAccLoad = (kPolicy & 2u) != 0;
  constexpr uint32_t kAccStore = acc_store<Op, FWD, WB, T>(), kOutStore = out_store<Op, FWD, WB, T>();
  constexpr uint32_t kUnit = 64u * U;
  const uint32_t nvec = len >> 4;
  const uint32_t v0 = trip * kUnit;
  const u32x4* rp = reinterpret_cast<const u32x4*>(r) + v0 + lane;
  u32x4* ap = reinterpret_cast<u32x4*>(a) + v0 + lane;
  u32x4* op = reinterpret_cast<u32x4*>(o) + v0 + lane;
  const StoreUnit<kAccStore, kUnit> kept(reinterpret_cast<u32x4*>(a) + v0, ap);
  const StoreUnit<kOutStore, kUnit> forwarded(reinterpret_cast<u32x4*>(o) + v0, op);
  if (v0 + kUnit <= nvec) {
    u32x4 rv[U], av[U];
#pragma unroll
    for (int u = 0; u < U; ++u) rv[u] = load16<kNtRecv>(rp + u * 64);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if constexpr (Op::kReadsAcc) av[u] = load16<kNtAccLoad>(ap + u * 64);
      else av[u] = rv[u];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const u32x4 t = combine<Op>(av[u], rv[u]);
      if (WB) kept.put(u * 64, lane, t);
      if (FWD) forwarded.put(u * 64, lane, t);
    }
    return;
  }
  // last unit of the chunk: ragged
#pragma unroll
  for (int u = 0; u < U; ++u) {
    if (v0 + lane + u * 64 < nvec) {
      const u32x4 rv = load16<kNtRecv>(rp + u * 64);
      u32x4 av = rv;
      if constexpr (Op::kReadsAcc) av = load16<kNtAccLoad>(ap + u * 64);
      const u32x4 t = combine<Op>(av, rv);
      if (WB) kept.put(u * 64, lane, t);
      if (FWD) forwarded.put(u * 64, lane, t);
    }
  }
  const uint32_t rem = len & 15u;
  if (rem) {  // nvec lies in this unit, or the chunk would have had one unit fewer
    const uint64_t off = static_cast<uint64_t>(nvec) << 4;
    stream_tail<Op, FWD, WB>(r + off, a + off, FWD ? o + off : o, rem, lane);
  }
}

// Whether the record's written streams begin on lines (the accumulator's place counts also where it is not kept).
__device__ __forceinline__ bool record_on_lines(const Args& g, uint64_t dst, uint64_t out) {
  return on_lines(g.acc + dst, out == UCCL_NO_FORWARD ? nullptr : g.out + (out & ~UCCL_FORWARD_ONLY));
}

// The winners' units are numbered consecutively across the tile and dealt round-robin to the
// wavefronts of the workgroup, so the machine sees the same stream whether a tile holds one
// 128 KiB chunk or thirty-two 4 KiB chunks.
template <int NT, int T, int U, class Op, Through H>
__global__ void __launch_bounds__(NT) chunk_flat_kernel(const Args g) {
  constexpr uint32_t kUnit = 64u * U;
  constexpr uint32_t kWaves = NT / 64;
  __shared__ Tile<T> s;
  const uint32_t tid = threadIdx.x;
  // Consecutive workgroups run on different XCDs (each with an L2 of its own) and take consecutive
  // tiles, so at any moment the whole chip works on one contiguous window of receive slots.  The
  // alternative, one contiguous eighth of the tiles per XCD, keeps records and bitmap words inside
  // one L2 but makes the chip work on eight distant windows at once: measured slower (build switch).
  uint32_t tile = blockIdx.x;
  if (UCCL_XCD_CONTIGUOUS) {
    const uint32_t per_xcd = (gridDim.x + 7u) / 8u;   // the launch has 8 * per_xcd workgroups
    tile = (blockIdx.x & 7u) * per_xcd + (blockIdx.x >> 3);
  }
  if (tid < 64) dedup_tile<T, Op, kUnit>(g, s, tile, tid);
  __syncthreads();

  const uint32_t count = s.count;
  const uint32_t total = s.first[count];
  const uint32_t wave = tid >> 6, lane = tid & 63u;
  for (uint32_t u = wave; u < total; u += kWaves) {
    uint32_t w = 0;
    if (T > 1) {
      const bool mine = lane < count && s.first[lane] <= u && u < s.first[lane + 1];
      w = __ffsll(static_cast<unsigned long long>(__ballot(mine))) - 1;  // exactly one lane
    }
    w = __builtin_amdgcn_readfirstlane(w);
    const uint32_t trip = u - __builtin_amdgcn_readfirstlane(s.first[w]);
    const uint64_t src = wave_uniform(s.src[w]);
    const uint64_t dst = wave_uniform(s.dst[w]);
    const uint64_t out = wave_uniform(s.out[w]);
    const uint32_t len = __builtin_amdgcn_readfirstlane(s.len[w]);
    if (out == UCCL_NO_FORWARD)
      stream_unit<U, Op, false, true, H>(g.recv + src, g.acc + dst, nullptr, len, trip, lane);
    else if (out & UCCL_FORWARD_ONLY)
      stream_unit<U, Op, true, false, H>(g.recv + src, g.acc + dst, g.out + (out & ~UCCL_FORWARD_ONLY), len, trip, lane);
    else
      stream_unit<U, Op, true, true, H>(g.recv + src, g.acc + dst, g.out + out, len, trip, lane);
  }
}

// ---- large calls: decide first, then stream in destination order ------------------------------
//
// What bounds a call of hundreds of MiB is how well the memory system takes its mix of reads and
// writes, and that depends on the order of the accesses.  Arrival order scatters two of the four
// streams (accumulator and staging) over the reorder window.  Measured with dense kernels of two reads
// and two writes, 240 MiB per stream: destinations scattered in 32 KiB blocks 5.4 TB/s, in order 5.8;
// in order, one 4 KiB block per 256-thread workgroup, at most 24 wavefronts per compute unit, 6.3; the
// read of the slots scattered instead of the destinations, 6.3 as well.  So such a call is two launches:
//
//   order    one lane per record validates it, a wavefront decides its 64 sequence numbers (decide_wave), and
//            the lane of a first arrival leaves its index in entry seq mod n of a table in scratch memory (an
//            atomic exchange; n = records of the launch).  Sequence numbers ascend with the destination
//            in a collective's stream and a call covers about one run of them, so the table lists the
//            winners in destination order.  Two winners of one entry (sequence numbers that are no run)
//            are both served: the one that was there moves to a second list, to the entry of its own index.
//   stream   workgroup b takes 4 KiB part b mod `parts` of the record in entry b / parts: no atomic, no
//            barrier, no LDS.  Consecutive workgroups run on different XCDs; runs of kOrderRun of them
//            (128 KiB) are laid out so that each XCD works on one contiguous piece (1 GiB reduce-scatter
//            590 us without, 562 us with it; 64 KiB 566, 256 KiB 565, 512 KiB 570).  A launch that
//            combines is held to six workgroups per compute unit by asking for 24 KiB of LDS that it does
//            not use (562 us; eight 609, seven 591, five 591); copies are not (the 256 MiB bf16 step: 269 us
//            either way; five 283).
//
// Words of both lists carry the call's tag as claim words do, so nothing is cleared.
// Entry i of the table is word 2 i and entry i of the second list word 2 i + 1: one load serves both.  (That list
// needs no atomics and spreads over all workgroups: with windows of 256 sequence numbers of which 64 are used three
// records of four are on it; numbered by a counter instead, 16 383 records of 16 KiB take 229 us, so 209.)  An entry
// also says whether its record has no more than one, two or four parts, so that a workgroup whose part
// does not exist leaves without reading the record.  Which of an entry's workgroups takes which part turns
// with the entry: records shorter than `parts` parts would otherwise leave the same workgroups idle every time,
// and as workgroups are dealt to the shader engines in turn, the same engines (5000 records of 4 KiB each
// in four parts: 73 us the two phases without, 47 with it).
constexpr uint32_t kOrderThreads = 256;            // 4 KiB per stream: one vector per lane
constexpr uint32_t kOrderPartBytes = kOrderThreads * 16u;
constexpr uint32_t kOrderRun = 32;
constexpr uint32_t kOrderReduceLds = 24576;

struct OrderArgs {
  unsigned long long* words;    // 2 * n_descs words: tag << 16 | size class << 14 | record
  unsigned long long tag;
};

// Record k (below 2^14), a first arrival, into the table of a launch of n records.
__device__ __forceinline__ void order_put(const OrderArgs& t, uint32_t n, uint32_t seq, uint32_t k, uint32_t len) {
  const uint32_t size = len <= kOrderPartBytes ? 0u : len <= 2u * kOrderPartBytes ? 1u : len <= 4u * kOrderPartBytes ? 2u : 3u;
  const unsigned long long was = __hip_atomic_exchange(t.words + 2u * static_cast<size_t>(seq % n), (t.tag << 16) | (size << 14) | k,
                                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if ((was >> 16) == t.tag) t.words[2u * (static_cast<size_t>(was) & 0x3FFFu) + 1u] = was;   // a record is displaced once at most
}

// Whether `entry` is of this call and its record has a part `part` (size class 3: any number of parts).
__device__ __forceinline__ bool order_has(const OrderArgs& t, unsigned long long entry, uint32_t part) {
  const uint32_t size = (static_cast<uint32_t>(entry) >> 14) & 3u;
  return (entry >> 16) == t.tag && (size == 3u || part < (1u << size));
}
__device__ __forceinline__ uint32_t order_record(unsigned long long entry) { return static_cast<uint32_t>(entry) & 0x3FFFu; }

// The n_descs * parts workgroups of a launch in the order of their work: workgroup b runs on XCD b mod 8.
__device__ __forceinline__ uint32_t order_position(uint32_t grid) {
  const uint32_t b = blockIdx.x, group = b / (8u * kOrderRun), in = b % (8u * kOrderRun);
  return (group + 1u) * (8u * kOrderRun) <= grid ? group * (8u * kOrderRun) + (in & 7u) * kOrderRun + (in >> 3) : b;
}

// ---- 64 sequence numbers at once ----------------------------------------------------------------
//
// An atomic of one lane costs its 128-byte line of the bitmap 3 - 5.5 ns, in which the line serves no other, and
// sequence numbers that arrive together lie on one or two lines: 1024 records whose lanes each ask for their own bit
// take 3.3 us, 10.5 us where neighbouring lanes ask for one word.  So a wavefront's lanes first meet in LDS: lanes
// with the same bitmap word OR their bits into one slot, the lane that opened the slot issues the slot's one atomic
// and leaves the old word there.  A lane's record is the first arrival if its lane was the first to set the bit in
// the slot and the old word has it clear, so of several lanes with one number exactly one can be.  A
// lane whose slot belongs to another word (words kDecideSlots apart) asks for itself, with the same instruction.
// The order launch between a bitmap fill and a streaming kernel adds to these, with the atomic per lane before / now:
// numbers scattered over a window of 1024 5.6 / 2.9 us, of 256 6.2 / 2.8, in order 10.9 / 2.7; 15 700 numbers at
// random over all of their words, where next to nothing meets, 7.0 / 7.4.  Eight wavefronts sharing slots leave the
// atomics fewer and the whole slower (3.6).
constexpr uint32_t kDecideSlots = 128;
struct DecideSlots {
  uint32_t word[kDecideSlots], bits[kDecideSlots], old[kDecideSlots];
};

// LDS between the lanes of one wavefront: its accesses are served in order, the compiler has to leave them so.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Run by all lanes of a wavefront, on slots of its own: whether the lane asks and its record is the first arrival of `seq`.
__device__ __forceinline__ bool decide_wave(DecideSlots& s, uint32_t* bitmap, bool asks, uint32_t seq, uint32_t lane) {
  constexpr uint32_t kNone = 0xFFFFFFFFu;   // no word's index: seq >> 5 stays below 2^27
#pragma unroll
  for (uint32_t i = 0; i < kDecideSlots; i += 64) {
    s.word[i + lane] = kNone;
    s.bits[i + lane] = 0u;
  }
  wave_sync();
  const uint32_t word = seq >> 5, bit = 1u << (seq & 31u), slot = word % kDecideSlots;
  bool opens = false, shares = false, first = false;
  if (asks) {
    const uint32_t was = atomicCAS(&s.word[slot], kNone, word);
    opens = was == kNone;
    shares = opens || was == word;
    if (shares) first = (atomicOr(&s.bits[slot], bit) & bit) == 0u;
  }
  wave_sync();
  uint32_t old = 0u;
  if (opens || (asks && !shares)) old = atomicOr(bitmap + word, opens ? s.bits[slot] : bit);
  if (opens) s.old[slot] = old;
  wave_sync();
  if (shares) return first && (s.old[slot] & bit) == 0u;
  return asks && (old & bit) == 0u;
}

template <uint32_t kEs>
__global__ void __launch_bounds__(kOrderThreads) chunk_order_kernel(const Args g, const OrderArgs t) {
  __shared__ DecideSlots s[kOrderThreads / 64];
  const uint32_t k = blockIdx.x * kOrderThreads + threadIdx.x;
  bool ok = false;
  uint32_t len = 0u, seq = 0u;
  if (k < g.n_descs) {
    const u32x4* p = reinterpret_cast<const u32x4*>(g.descs + k);
    const u32x4 lo = p[0], hi = p[1];
    const uint64_t src = lo.x | (static_cast<uint64_t>(lo.y) << 32);
    const uint64_t dst = lo.z | (static_cast<uint64_t>(lo.w) << 32);
    const uint64_t out = hi.x | (static_cast<uint64_t>(hi.y) << 32);
    len = hi.z;
    seq = hi.w;
    ok = record_ok<kEs>(g, src, dst, out, len, seq);
    if (!ok && g.rejected != nullptr) atomicAdd(g.rejected, 1u);
  }
  if (decide_wave(s[threadIdx.x >> 6], g.bitmap, ok, seq, threadIdx.x & 63u)) order_put(t, g.n_descs, seq, k, len);
}

// Part `part` of record k: units part * 4 + wavefront, then every parts * 4 units (a record longer
// than all its parts).  H: as a record's stores are written if it begins on lines, which is looked at here: one branch a part.
// (chunk_few_kernel does the same for records of unknown size; elsewhere the host chooses: a choice at each store costs 1.07 - 1.1 times there, one
// for a unit in chunk_flat_kernel's copies 2 % of 128 messages in 4 KiB chunks.)
template <class Op, Through H>
__device__ __forceinline__ void ordered_units(const Args& g, const uccl_chunk_desc& d, uint32_t part) {
  constexpr uint32_t kUnit = 64u, kWaves = kOrderThreads / 64;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63u;
  const uint32_t vecs = (d.len >> 4) + ((d.len & 15u) != 0u ? 1u : 0u);
  const uint32_t total = (vecs + kUnit - 1u) / kUnit;
  for (uint32_t u = part * kWaves + wave; u < total; u += g.parts * kWaves) {
    if (d.out_off == UCCL_NO_FORWARD)
      stream_unit<1, Op, false, true, H>(g.recv + d.src_off, g.acc + d.dst_off, nullptr, d.len, u, lane);
    else if (d.out_off & UCCL_FORWARD_ONLY)
      stream_unit<1, Op, true, false, H>(g.recv + d.src_off, g.acc + d.dst_off, g.out + (d.out_off & ~UCCL_FORWARD_ONLY), d.len, u, lane);
    else
      stream_unit<1, Op, true, true, H>(g.recv + d.src_off, g.acc + d.dst_off, g.out + d.out_off, d.len, u, lane);
  }
}
template <class Op, Through H>
__device__ __forceinline__ void ordered_part(const Args& g, uint32_t k, uint32_t part) {
  const uccl_chunk_desc d = g.descs[k];   // the same address in every lane
  if (H != kNoThrough && record_on_lines(g, d.dst_off, d.out_off)) ordered_units<Op, H>(g, d, part);
  else ordered_units<Op, kNoThrough>(g, d, part);
}

template <class Op, Through H>
__global__ void __launch_bounds__(kOrderThreads) chunk_ordered_kernel(const Args g, const OrderArgs t) {
  const uint32_t b = order_position(g.n_descs * g.parts), entry = b / g.parts, part = (b + entry) % g.parts;
  const unsigned long long first = t.words[2u * static_cast<size_t>(entry)];
  const unsigned long long second = t.words[2u * static_cast<size_t>(entry) + 1u];
  if (order_has(t, first, part)) ordered_part<Op, H>(g, order_record(first), part);
  if (order_has(t, second, part)) ordered_part<Op, H>(g, order_record(second), part);
}

// ---- calls of few records --------------------------------------------------------------------
//
// A call of a few dozen records (a 4 MiB message in 64 KiB chunks is 57 of them per phase) cannot
// fill the machine; what it costs is one workgroup's chain of latencies: read the record, decide
// the sequence number (one atomic round trip), read the payload, write it.  This kernel shortens
// the chain instead of the stream: one record per workgroup (or per group of `parts` workgroups),
// every wavefront reads the record for itself and issues the loads of its first unit at once,
// while one lane decides the sequence number; after one barrier the winners combine and store
// what is already in registers.  A duplicate therefore costs its payload reads (never a write),
// which is why calls of many records, where duplicates are many and latency is hidden by the
// number of workgroups anyway, use chunk_flat_kernel.  PARTS: blockIdx.x = record * parts + part
// (see claim_enter).
template <int U, class Op, bool FWD, bool WB, Through T>
__device__ __forceinline__ void finish_unit(const u32x4 (&rv)[U], const u32x4 (&av)[U], u32x4* au, u32x4* ou, u32x4* ap, u32x4* op, uint32_t lane,
                                            uint32_t first_vec, uint32_t nvec) {
  const StoreUnit<acc_store<Op, FWD, WB, T>(), 64u * U> kept(au, ap);
  const StoreUnit<out_store<Op, FWD, WB, T>(), 64u * U> forwarded(ou, op);
#pragma unroll
  for (int u = 0; u < U; ++u) {
    if (first_vec + u * 64 < nvec) {
      const u32x4 t = combine<Op>(Op::kReadsAcc ? av[u] : rv[u], rv[u]);
      if (WB) kept.put(u * 64, lane, t);
      if (FWD) forwarded.put(u * 64, lane, t);
    }
  }
}

// Waits for the wavefront's loads (vmcnt 0), once.  Left to itself the compiler waits in front of each vector that a lane may not
// have, and as loads and stores are counted together, that is for the store of the vector before: one that is written through takes its time
// (ring of 24 MiB bf16 in 32 KiB chunks, decided 64 at a time, 31.5 / 30.2 us; 40 MiB f32, a workgroup a record, 49.3 / 47.9).
__device__ __forceinline__ void await_loads() { __builtin_amdgcn_s_waitcnt(0x0F70); }

template <int NT, int U, class Op, Through H, bool PARTS, bool APART = false>
__global__ void __launch_bounds__(NT) chunk_few_kernel(const Args g) {
  constexpr uint32_t kUnit = 64u * U;
  constexpr uint32_t kWaves = NT / 64;
  __shared__ uint32_t s_win;
  const uint32_t tid = threadIdx.x, lane = tid & 63u;
  const uint32_t wave = H == kNoThrough ? tid >> 6 : __builtin_amdgcn_readfirstlane(tid >> 6);   // a scalar where units' places are
  const uint32_t k = PARTS ? blockIdx.x / g.parts : blockIdx.x;   // the launch has n_descs (* parts) workgroups
  const uint32_t part = PARTS ? blockIdx.x % g.parts : 0u;

  unsigned long long* const claim = PARTS ? g.claims + static_cast<size_t>(k) * UCCL_CLAIM_STRIDE : nullptr;

  // every lane reads the same 32 bytes: one request per wavefront
  const u32x4* p = reinterpret_cast<const u32x4*>(g.descs + k);
  const u32x4 lo = p[0], hi = p[1];
  const uint32_t live = g.n_ptr != nullptr ? *g.n_ptr : g.n_descs;
  const uint64_t src = wave_uniform(lo.x | (static_cast<uint64_t>(lo.y) << 32));
  const uint64_t dst = wave_uniform(lo.z | (static_cast<uint64_t>(lo.w) << 32));
  const uint64_t out = wave_uniform(hi.x | (static_cast<uint64_t>(hi.y) << 32));
  const uint32_t len = __builtin_amdgcn_readfirstlane(hi.z);
  const uint32_t seq = __builtin_amdgcn_readfirstlane(hi.w);
  const bool is_record = k < live;
  const bool ok = is_record && record_ok<Op::kEs>(g, src, dst, out, len, seq);

  const uint32_t nvec = len >> 4;
  const uint32_t vecs = nvec + ((len & 15u) != 0u ? 1u : 0u);
  const uint32_t total = (vecs + kUnit - 1u) / kUnit;
  const uint32_t stride = PARTS ? kWaves * g.parts : kWaves;
  const uint32_t u0 = part * kWaves + wave;
  const uint32_t first_vec = u0 * kUnit + lane;
  const bool have = ok && u0 < total;
  const bool part_has_units = ok && part * kWaves < total;  // uniform over the workgroup
  const u32x4* rp = reinterpret_cast<const u32x4*>(g.recv + src) + first_vec;
  u32x4* ap = reinterpret_cast<u32x4*>(g.acc + dst) + first_vec;
  u32x4 rv[U], av[U];
  if (have) {  // in bounds whether or not this record turns out to be the first arrival
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (first_vec + u * 64 < nvec) rv[u] = __builtin_nontemporal_load(rp + u * 64);
    if constexpr (Op::kReadsAcc) {
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (first_vec + u * 64 < nvec) av[u] = ap[u * 64];
    }
  }
  if (tid == 0) {
    uint32_t win = 0u;
    Claim entered = {true, 0ull};
    if constexpr (PARTS) entered = claim_enter<APART>(claim, g.tag);
    if (entered.decides) {
      if (ok) {
        const uint32_t bit = 1u << (seq & 31u);
        win = (atomicOr(g.bitmap + (seq >> 5), bit) & bit) == 0u ? 1u : 0u;
      } else if (is_record && g.rejected != nullptr) {  // a rejected record is counted once: by the part that decides
        atomicAdd(g.rejected, 1u);
      }
      if constexpr (PARTS) claim_publish<APART>(claim, g.tag, win != 0u);
    } else if (part_has_units) {  // a part without units has nothing to wait for
      win = claim_await<APART>(claim, entered.seen, g.tag, g.faults()) ? 1u : 0u;
    }
    s_win = win;
  }
  __syncthreads();
  if (s_win == 0u) return;
  const bool fwd = out != UCCL_NO_FORWARD;
  const bool relay = fwd && (out & UCCL_FORWARD_ONLY) != 0;
  char* const o = g.out + (out & ~UCCL_FORWARD_ONLY);
  const auto finish = [&](auto how) {
    constexpr Through kHow = decltype(how)::value;
    if constexpr (kHow != kNoThrough) await_loads();
    if (have) {
      u32x4* op = reinterpret_cast<u32x4*>(o) + first_vec;
      u32x4* const au = reinterpret_cast<u32x4*>(g.acc + dst) + u0 * kUnit;
      u32x4* const ou = reinterpret_cast<u32x4*>(o) + u0 * kUnit;
      if (!fwd) finish_unit<U, Op, false, true, kHow>(rv, av, au, ou, ap, op, lane, first_vec, nvec);
      else if (relay) finish_unit<U, Op, true, false, kHow>(rv, av, au, ou, ap, op, lane, first_vec, nvec);
      else finish_unit<U, Op, true, true, kHow>(rv, av, au, ou, ap, op, lane, first_vec, nvec);
      const uint32_t rem = len & 15u;
      if (rem != 0u && nvec >= u0 * kUnit && nvec < (u0 + 1u) * kUnit) {  // the unit that holds the partial vector
        const uint64_t off = static_cast<uint64_t>(nvec) << 4;
        if (!fwd) stream_tail<Op, false, true>(g.recv + src + off, g.acc + dst + off, nullptr, rem, lane);
        else if (relay) stream_tail<Op, true, false>(g.recv + src + off, g.acc + dst + off, o + off, rem, lane);
        else stream_tail<Op, true, true>(g.recv + src + off, g.acc + dst + off, o + off, rem, lane);
      }
    }
    for (uint32_t u = u0 + stride; u < total; u += stride) {
      if (!fwd) stream_unit<U, Op, false, true, kHow>(g.recv + src, g.acc + dst, nullptr, len, u, lane);
      else if (relay) stream_unit<U, Op, true, false, kHow>(g.recv + src, g.acc + dst, o, len, u, lane);
      else stream_unit<U, Op, true, true, kHow>(g.recv + src, g.acc + dst, o, len, u, lane);
    }
  };
  // The size not stated: the record's own says whether the call is likely to be small.  One choice between two bodies costs nothing to speak of; one at
  // each store costs records that are long 7 - 10 %, as the loads of their later units no longer overlap.
  if constexpr (H != kByRecord) finish(Stores<H>());
  else if (static_cast<uint64_t>(len) * g.n_descs <= kThroughBytes || record_on_lines(g, dst, out)) finish(Stores<kAllThrough>());
  else finish(Stores<kNoThrough>());
}

// ---- calls of hundreds of records -------------------------------------------------------------------
//
// With a workgroup per record that decides for itself, the atomics of n single lanes meet on one or two lines of the
// bitmap, some 6.5 ns each; tiles of records have few atomics but leave compute units idle below some 4000
// records.  Here a workgroup takes one record (or one of `parts` parts of it) and loads its payload at
// once, but records are decided kGroup at a time (decide_wave), by the first wavefront of the group's first
// workgroup; the others poll for the outcome, which comes at about the time their payload does.  What is left is the
// chain record, LDS, atomic OR, outcome, payload store.  Measured, us a pass of reset, SUM with forward and COPY with
// forward, before / now: 949 x 5.7 KB of unknown size 25.3 / 14.2; 4 KiB chunks 320 records 12.6 / 10.8,
// 1280 19.4 / 15.7, 2560 28.2 / 25.8; 640 x 8 KiB 18.1 / 15.2; 640 x 16 KiB 26.2 / 20.9; 320 x 128 KiB 64.8 / 56.2.
//
// A group's line of scratch words holds a claim word and its outcome, a bit per record in four words, all as
// `tag << 16 | value`.  A wavefront that has polled kGroupPolls times exchanges the claim word as well and decides if the
// first workgroup has not begun to; so everyone waits for a wavefront that is running and waits for nobody, and the
// wait ends whatever order the hardware starts workgroups in.  It is bounded all the same, as in claim_await.
//
// Not for larger calls: each round of workgroups that the chip holds waits for its decisions once more (10 240 x 4 KiB
// 62 / 78 us; deciding a round ahead takes 63, and gives smaller calls nothing).
#ifndef UCCL_GROUP_POLLS
#define UCCL_GROUP_POLLS 4096
#endif
#ifndef UCCL_GROUP_LEADS
#define UCCL_GROUP_LEADS 1      // tests' builds: 0 the group's first workgroup waits like the others, 2 it comes late
#endif
constexpr uint32_t kGroup = 64;
constexpr uint32_t kGroupPolls = UCCL_GROUP_POLLS;

// Lane 0 asks to decide the group; what the claim word held says whether it may (group_is_ours).
__device__ __forceinline__ unsigned long long group_enter(unsigned long long* line, unsigned long long tag, uint32_t lane) {
  unsigned long long was = 0ull;
  if (lane == 0) was = __hip_atomic_exchange(line, tag << 16, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return was;
}
// What the leader does first.  Nothing; in a test's build it waits for another to begin to decide (not for long: there may be none).
__device__ __forceinline__ void group_lead(unsigned long long* line, unsigned long long tag) {
#if UCCL_GROUP_LEADS == 2
  for (uint32_t polls = 0; polls < 4096u && (__hip_atomic_load(line, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> 16) != tag; ++polls)
    __builtin_amdgcn_s_sleep(1);
#endif
}
__device__ __forceinline__ bool group_is_ours(unsigned long long was, unsigned long long tag) {
  return __builtin_amdgcn_readfirstlane(static_cast<uint32_t>((was >> 16) != tag)) != 0u;
}
__device__ __forceinline__ void group_publish(unsigned long long* line, unsigned long long tag, unsigned long long outcome, uint32_t lane) {
  if (lane < 4u)
    __hip_atomic_store(line + 1u + lane, (tag << 16) | ((outcome >> (16u * lane)) & 0xFFFFull), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Whether record `in` of the group is a first arrival.  By all lanes of a workgroup's first wavefront.  `decides`: it
// has entered first, and found `was`.  `waits`: it has a use for the answer.  again(): the group's records are read (a
// later claim).  decide(): the ballot of their first arrivals.
template <class Again, class Decide>
__device__ __forceinline__ bool group_outcome(unsigned long long* line, unsigned long long tag, unsigned long long was, bool decides, bool waits,
                                              uint32_t in, uint32_t lane, uint32_t* faults, Again again, Decide decide) {
  for (uint32_t polls = 0;; ++polls) {
    if (decides || polls == kGroupPolls) {
      if (!decides) {
        was = group_enter(line, tag, lane);
        again();
      }
      decides = false;
      if (group_is_ours(was, tag)) {
        const unsigned long long outcome = decide();
        group_publish(line, tag, outcome, lane);
        return ((outcome >> in) & 1ull) != 0ull;
      }
    }
    if (!waits) return false;
    unsigned long long seen = 0ull;
    if (lane == 0) seen = __hip_atomic_load(line + 1u + (in >> 4), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (!group_is_ours(seen, tag)) return ((__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(seen)) >> (in & 15u)) & 1u) != 0u;
    if (polls >= UCCL_CLAIM_SPIN_LIMIT) {
      if (lane == 0) atomicAdd(faults, 1u);
      return false;
    }
    __builtin_amdgcn_s_sleep(1);
  }
}

// Workgroup b's record and part.  Records whose size is stated come one after the other, so that the chip works on one
// window of the payload; the parts turn with the record (see order_position).  Where it is not, most parts may have nothing to
// do, so part 0 of every record comes first and the others after it (PART_MAJOR): what a short record does not need is then
// launched when the payload of all is on its way (1280 records of unknown size in two parts, 4 / 32 / 64 KiB, us a pass: record
// by record 11.8 / 31.9 / 55.1, this way 8.7 / 31.0 / 54.9, one part 8.7 / 30.2 / 54.7).
struct GroupPlace {
  uint32_t k, part, in, base;   // record, part, and the record's place in its group, which begins at `base`
  bool first;                   // the first workgroup of the group that is launched
};
template <bool PART_MAJOR>
__device__ __forceinline__ GroupPlace group_place(const ClaimArgs& g) {
  GroupPlace p;
  p.k = PART_MAJOR ? blockIdx.x % g.n_descs : blockIdx.x / g.parts;
  p.part = PART_MAJOR ? blockIdx.x / g.n_descs : (blockIdx.x + p.k) % g.parts;
  p.in = p.k % kGroup;
  p.base = p.k - p.in;
  p.first = blockIdx.x == (PART_MAJOR ? p.base : p.base * g.parts);
  return p;
}

template <int NT, int U, class Op, bool PART_MAJOR, Through H>
__global__ void __launch_bounds__(NT) UCCL_FULL_OCCUPANCY chunk_group_kernel(const Args g) {
  constexpr uint32_t kUnit = 64u * U;
  constexpr uint32_t kWaves = NT / 64;
  __shared__ DecideSlots s;
  __shared__ uint32_t s_win;
  const uint32_t tid = threadIdx.x, lane = tid & 63u;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const GroupPlace place = group_place<PART_MAJOR>(g);   // the launch has n_descs * parts workgroups
  const uint32_t k = place.k, part = place.part, in = place.in, base = place.base;
  const bool decides = UCCL_GROUP_LEADS && wave == 0u && place.first;
  unsigned long long* const line = g.claims + static_cast<size_t>(base / kGroup) * UCCL_CLAIM_STRIDE;
  unsigned long long was = 0ull;
  if (decides) {
    group_lead(line, g.tag);
    was = group_enter(line, g.tag, lane);
  }
  // every lane reads the workgroup's record; where the group is decided, lane i reads record i of the group
  const uint32_t mine = decides && base + lane < g.n_descs ? base + lane : k;
  const u32x4* p = reinterpret_cast<const u32x4*>(g.descs + mine);
  u32x4 lo = p[0], hi = p[1];
  const uint64_t src = wave_uniform(lo.x | (static_cast<uint64_t>(lo.y) << 32));   // of lane 0: that is record k in either case
  const uint64_t dst = wave_uniform(lo.z | (static_cast<uint64_t>(lo.w) << 32));
  const uint64_t out = wave_uniform(hi.x | (static_cast<uint64_t>(hi.y) << 32));
  const uint32_t len = __builtin_amdgcn_readfirstlane(hi.z);
  const bool ok = record_ok<Op::kEs>(g, src, dst, out, len, __builtin_amdgcn_readfirstlane(hi.w));

  const uint32_t nvec = len >> 4;
  const uint32_t vecs = nvec + ((len & 15u) != 0u ? 1u : 0u);
  const uint32_t total = (vecs + kUnit - 1u) / kUnit;
  const uint32_t stride = kWaves * g.parts;
  const uint32_t u0 = part * kWaves + wave;
  const uint32_t first_vec = u0 * kUnit + lane;
  const bool have = ok && u0 < total;
  const bool part_has_units = ok && part * kWaves < total;  // uniform over the workgroup
  const u32x4* rp = reinterpret_cast<const u32x4*>(g.recv + src) + first_vec;
  u32x4* ap = reinterpret_cast<u32x4*>(g.acc + dst) + first_vec;
  u32x4 rv[U], av[U];
  const auto load = [&] {   // in bounds whether or not this record turns out to be the first arrival
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (first_vec + u * 64 < nvec) rv[u] = __builtin_nontemporal_load(rp + u * 64);
    if constexpr (Op::kReadsAcc) {
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (first_vec + u * 64 < nvec) av[u] = ap[u * 64];
    }
  };
  if (have && !decides) load();
  if (wave == 0u) {
    const bool win = group_outcome(
        line, g.tag, was, decides, part_has_units, in, lane, g.faults(),
        [&] {
          const u32x4* q = reinterpret_cast<const u32x4*>(g.descs + (base + lane < g.n_descs ? base + lane : k));
          lo = q[0];
          hi = q[1];
        },
        [&] {
          const bool is_record = base + lane < g.n_descs;
          const bool good = is_record && record_ok<Op::kEs>(g, lo.x | (static_cast<uint64_t>(lo.y) << 32), lo.z | (static_cast<uint64_t>(lo.w) << 32),
                                                            hi.x | (static_cast<uint64_t>(hi.y) << 32), hi.z, hi.w);
          if (is_record && !good && g.rejected != nullptr) atomicAdd(g.rejected, 1u);
          return __ballot(decide_wave(s, g.bitmap, good, hi.w, lane));
        });
    if (have && decides) load();   // memory operations return in order: issued earlier, they would hold up the decision
    if (lane == 0) s_win = win ? 1u : 0u;
  }
  if (!part_has_units) return;   // the whole workgroup
  __syncthreads();
  if (s_win == 0u) return;
  const bool fwd = out != UCCL_NO_FORWARD;
  const bool relay = fwd && (out & UCCL_FORWARD_ONLY) != 0;
  char* const o = g.out + (out & ~UCCL_FORWARD_ONLY);
  if constexpr (H != kNoThrough) await_loads();
  if (have) {
    u32x4* op = reinterpret_cast<u32x4*>(o) + first_vec;
    u32x4* const au = reinterpret_cast<u32x4*>(g.acc + dst) + u0 * kUnit;
    u32x4* const ou = reinterpret_cast<u32x4*>(o) + u0 * kUnit;
    if (!fwd) finish_unit<U, Op, false, true, H>(rv, av, au, ou, ap, op, lane, first_vec, nvec);
    else if (relay) finish_unit<U, Op, true, false, H>(rv, av, au, ou, ap, op, lane, first_vec, nvec);
    else finish_unit<U, Op, true, true, H>(rv, av, au, ou, ap, op, lane, first_vec, nvec);
    const uint32_t rem = len & 15u;
    if (rem != 0u && nvec >= u0 * kUnit && nvec < (u0 + 1u) * kUnit) {  // the unit that holds the partial vector
      const uint64_t off = static_cast<uint64_t>(nvec) << 4;
      if (!fwd) stream_tail<Op, false, true>(g.recv + src + off, g.acc + dst + off, nullptr, rem, lane);
      else if (relay) stream_tail<Op, true, false>(g.recv + src + off, g.acc + dst + off, o + off, rem, lane);
      else stream_tail<Op, true, true>(g.recv + src + off, g.acc + dst + off, o + off, rem, lane);
    }
  }
  for (uint32_t u = u0 + stride; u < total; u += stride) {
    if (!fwd) stream_unit<U, Op, false, true, H>(g.recv + src, g.acc + dst, nullptr, len, u, lane);
    else if (relay) stream_unit<U, Op, true, false, H>(g.recv + src, g.acc + dst, o, len, u, lane);
    else stream_unit<U, Op, true, true, H>(g.recv + src, g.acc + dst, o, len, u, lane);
  }
}

// ---- several sources per destination chunk ---------------------------------------------
//
// Section 2.1: the kernel reduces transport buffers "from multiple sender GPUs" into the
// tensor buffer.  A gather record names up to UCCL_MAX_SOURCES receive slots for one
// destination chunk; they are folded into the accumulator's value in the order listed, so
// the floating-point result is fixed by the record, not by arrival timing.  The accumulator
// is read and written once per chunk however many sources there are.  Same tile / unit
// dealing as chunk_flat_kernel; per unit a wavefront keeps the running value in registers
// (widened to binary32 for 16-bit types); sources are loaded in batches, all loads of a
// batch in flight before the folds, which then run in the listed order.
struct GatherArgs : Buffers<uccl_gather_desc>, ClaimArgs {};
static_assert(sizeof(GatherArgs) <= 112, "see ClaimArgs");

// What a record must satisfy but for its sources, and what each of them must.
template <uint32_t kEs>
__device__ __forceinline__ bool gather_ok(const GatherArgs& g, uint64_t dst, uint64_t out, uint32_t len, uint32_t seq, uint32_t n_src) {
  const uint64_t out_at = out & ~UCCL_FORWARD_ONLY;
  bool ok = seq < g.ext.n_bits && (dst & 15u) == 0 && len % kEs == 0 && n_src >= 1 && n_src <= UCCL_MAX_SOURCES &&
            dst <= g.ext.acc_bytes && len <= g.ext.acc_bytes - dst;
  if (out != UCCL_NO_FORWARD)
    ok = ok && g.out != nullptr && (out_at & 15u) == 0 && out_at <= g.ext.out_bytes && len <= g.ext.out_bytes - out_at;
  return ok;
}
__device__ __forceinline__ bool gather_source_ok(const GatherArgs& g, uint64_t src, uint32_t len) {
  return (src & 15u) == 0 && src <= g.ext.recv_bytes && len <= g.ext.recv_bytes - src;
}

// All sources of the lane's record, eight at a time: the offsets are loaded together whether they are named or not (a record
// has room for all) and checked after, for one latency instead of one per source (140 x 4 KiB from 16 sources decided
// 64 records at a time 11.2 / 9.3 us, 600 x 8 KiB from seven 13.9 / 12.9).
__device__ __forceinline__ bool gather_sources_ok(const GatherArgs& g, const uccl_gather_desc* d, uint32_t n_src, uint32_t len) {
  bool ok = true;
#pragma unroll
  for (uint32_t half = 0; half < UCCL_MAX_SOURCES; half += 8) {
    if (n_src > half) {
      const u32x4* p = reinterpret_cast<const u32x4*>(d->src_off + half);
      u32x4 v[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = p[i];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint64_t a = v[i].x | (static_cast<uint64_t>(v[i].y) << 32), b = v[i].z | (static_cast<uint64_t>(v[i].w) << 32);
        if (half + 2 * i < n_src) ok = ok && gather_source_ok(g, a, len);
        if (half + 2 * i + 1 < n_src) ok = ok && gather_source_ok(g, b, len);
      }
    }
  }
  return ok;
}

// One unit (64 * U vectors from vector v0 on) of one destination chunk: the accumulator's value and the
// sources folded into it in the listed order (fold), the result written back and / or forwarded (store).
// Sources are loaded in batches of B, all loads of a batch issued before the folds.  src(j): offset of
// source j, the same in every lane.  ACC: how the result is stored.  Through, us a pass, default policy / this: tiles 60 MiB
// in 4 KiB chunks from three sources 62.3 / 58.8, 64 MiB in 9 008-byte ones from two 53.9 / 52.3; decided 64 at a time 20 MiB in 64 KiB chunks from seven 36.8 / 35.5,
// 30 MiB in 6 000-byte ones 63.3 / 60.7; in destination order 128 MiB in 128 KiB chunks from seven 206 / 197, 100 MiB in 20 000-byte ones from three 104.6 / 99.4.
// Where a line is two chunks' it goes out in parts: tiles of chunks that are no whole lines lose from one source once they have left the last-level cache, 100 MiB in 9 008-byte chunks
// 68.8 / 72.3, 200 MiB 133.5 / 137.4, in 6 000 136.6 / 137.7, in 12 400 134.4 / 135.8, from three 217.7 / 218.2, from seven (100 MiB) 197.9 / 195.0; the host does not know how many there are, so above 72 MiB they keep the
// default policy.  Of unknown size all is written through, which costs such calls from one source 3 % (200 MiB in 9 008 133.7 / 137.8, 250 MiB in 33 008 176 / 182; 70 MiB 42.9 / 42.0): choosing
// by the tile's first record in the kernel costs those in whole lines 2 % (200 MiB in 4 KiB chunks 129.9 / 132.3, default 131.2), choosing at the store 12 %.
// Calls cut into parts keep the default policy: they are over before there is much to write back (1.8 MiB from two sources 7.1 / 7.6).
// Never non-temporally: a fold's result has a reader.  In destination order the call alone would take less, with uccl_chunk_segment of the result after it
// more, default policy / through / through and non-temporal: 128 MiB from one source 74.5 / 72.0 / 69.8, with it 110.9 / 108.1 / 115.9; from seven 206 / 197 / 190, 244.6 / 235.3 / 237.7;
// 96 MiB from one 58.1 / 56.3 / 54.4, 84.1 / 82.6 / 88.2; 256 MiB bf16 from two 189 / 185 / 182, 261 / 257 / 278.  The forwarded copy is non-temporal, as it was.
template <int U, class Op>
struct GatherUnit {
  bool live[U];
  typename Op::State st[U][4];
};

template <int U, int B, class Op, class Src>
__device__ __forceinline__ void gather_fold(const GatherArgs& g, GatherUnit<U, Op>& t, uint64_t dst, uint32_t len, uint32_t n_src, Src src,
                                            uint32_t v0, uint32_t lane) {
  const uint32_t nvec = len >> 4;
  const u32x4* ap = reinterpret_cast<const u32x4*>(g.acc + dst) + v0 + lane;
#pragma unroll
  for (int i = 0; i < U; ++i) {
    t.live[i] = v0 + lane + i * 64 < nvec;
    u32x4 a = {0u, 0u, 0u, 0u};
    if (t.live[i]) a = ap[i * 64];
    t.st[i][0] = Op::open(a.x); t.st[i][1] = Op::open(a.y); t.st[i][2] = Op::open(a.z); t.st[i][3] = Op::open(a.w);
  }
  for (uint32_t j0 = 0; j0 < n_src; j0 += B) {
    u32x4 rv[B][U];
#pragma unroll
    for (uint32_t b = 0; b < B; ++b) {
      if (j0 + b < n_src) {
        const u32x4* rp = reinterpret_cast<const u32x4*>(g.recv + src(j0 + b)) + v0 + lane;
#pragma unroll
        for (int i = 0; i < U; ++i) {
          rv[b][i] = u32x4{0u, 0u, 0u, 0u};
          if (t.live[i]) rv[b][i] = __builtin_nontemporal_load(rp + i * 64);
        }
      }
    }
#pragma unroll
    for (uint32_t b = 0; b < B; ++b) {
      if (j0 + b < n_src) {
#pragma unroll
        for (int i = 0; i < U; ++i) {
          Op::fold(t.st[i][0], rv[b][i].x); Op::fold(t.st[i][1], rv[b][i].y);
          Op::fold(t.st[i][2], rv[b][i].z); Op::fold(t.st[i][3], rv[b][i].w);
        }
      }
    }
  }
}

template <int U, uint32_t ACC, class Op, class Src>
__device__ __forceinline__ void gather_store(const GatherArgs& g, const GatherUnit<U, Op>& u, uint64_t dst, uint64_t out, uint32_t len,
                                             uint32_t n_src, Src src, uint32_t v0, uint32_t lane) {
  static_assert(ACC == kCached || ACC == kThrough, "kept for the result's reader");
  constexpr uint32_t kUnit = 64u * U;
  const uint32_t nvec = len >> 4;
  const bool fwd = out != UCCL_NO_FORWARD;
  const bool keep = !(fwd && (out & UCCL_FORWARD_ONLY));
  u32x4* au = reinterpret_cast<u32x4*>(g.acc + dst) + v0;
  u32x4* ou = reinterpret_cast<u32x4*>(g.out + (out & ~UCCL_FORWARD_ONLY)) + v0;
  const StoreUnit<ACC, kUnit> kept(au, au + lane);
  const StoreUnit<kOnce, kUnit> forwarded(ou, ou + lane);
#pragma unroll
  for (int i = 0; i < U; ++i) {
    if (!u.live[i]) continue;
    u32x4 t;
    t.x = Op::close(u.st[i][0]); t.y = Op::close(u.st[i][1]); t.z = Op::close(u.st[i][2]); t.w = Op::close(u.st[i][3]);
    if (keep) kept.put(i * 64, lane, t);
    if (fwd) forwarded.put(i * 64, lane, t);
  }
  // the last len % 16 bytes, element by element, by the unit that holds vector index nvec.  The whole wavefront walks
  // the sources (src may read another lane's register); only the loads and stores are the lanes' that have an element.
  const uint32_t rem = len & 15u;
  if (rem && nvec >= v0 && nvec < v0 + kUnit) {
    const bool mine = lane < rem / Op::kEs;
    const uint64_t off = (static_cast<uint64_t>(nvec) << 4) + lane * Op::kEs;
    uint32_t a_el = 0u;
    if (mine) {
      if constexpr (Op::kEs == 4) a_el = *reinterpret_cast<const uint32_t*>(g.acc + dst + off);
      else a_el = *reinterpret_cast<const uint16_t*>(g.acc + dst + off);
    }
    typename Op::State t = Op::open(a_el);
    for (uint32_t j = 0; j < n_src; ++j) {
      const char* rp = g.recv + src(j) + off;
      uint32_t r_el = 0u;
      if (mine) {
        if constexpr (Op::kEs == 4) r_el = *reinterpret_cast<const uint32_t*>(rp);
        else r_el = *reinterpret_cast<const uint16_t*>(rp);
      }
      Op::fold(t, r_el);
    }
    const uint32_t res = Op::close(t);
    if (mine) {
      if constexpr (Op::kEs == 4) {
        if (keep) *reinterpret_cast<uint32_t*>(g.acc + dst + off) = res;
        if (fwd) *reinterpret_cast<uint32_t*>(g.out + (out & ~UCCL_FORWARD_ONLY) + off) = res;
      } else {
        if (keep) *reinterpret_cast<uint16_t*>(g.acc + dst + off) = static_cast<uint16_t>(res);
        if (fwd) *reinterpret_cast<uint16_t*>(g.out + (out & ~UCCL_FORWARD_ONLY) + off) = static_cast<uint16_t>(res);
      }
    }
  }
}

// Both, with the sources' offsets in memory (src[], the same address in every lane).
template <int U, uint32_t ACC, class Op>
__device__ __forceinline__ void gather_unit(const GatherArgs& g, uint64_t dst, uint64_t out, uint32_t len,
                                            uint32_t n_src, const uint64_t* src, uint32_t v0, uint32_t lane) {
  const auto at = [src](uint32_t j) { return wave_uniform(src[j]); };
  GatherUnit<U, Op> t;
  gather_fold<U, UCCL_GATHER_BATCH, Op>(g, t, dst, len, n_src, at, v0, lane);
  gather_store<U, ACC, Op>(g, t, dst, out, len, n_src, at, v0, lane);
}

template <int T>
struct GatherTile {
  uint64_t dst[T], out[T];
  uint64_t src[T][UCCL_MAX_SOURCES];
  uint32_t len[T], n_src[T];
  uint32_t first[T + 1];
  uint32_t count;
};

template <int NT, int T, int U, class Op, Store ACC>
__global__ void __launch_bounds__(NT) chunk_gather_kernel(const GatherArgs g) {
  static_assert(T >= 1 && T <= 64, "one wavefront dedups the tile");
  constexpr uint32_t kUnit = 64u * U;
  __shared__ GatherTile<T> s;
  const uint32_t tid = threadIdx.x;
  if (tid < 64) {
    const uint64_t k = static_cast<uint64_t>(blockIdx.x) * T + tid;
    bool win = false;
    uint64_t dst = 0, out = 0;
    uint32_t len = 0, n_src = 0;
    const uccl_gather_desc* d = g.descs + k;
    if (tid < T && k < g.n_descs) {
      const u32x4* p = reinterpret_cast<const u32x4*>(d);
      const u32x4 lo = p[0], hi = p[1];
      dst = lo.x | (static_cast<uint64_t>(lo.y) << 32);
      out = lo.z | (static_cast<uint64_t>(lo.w) << 32);
      len = hi.x;
      const uint32_t seq = hi.y;
      n_src = hi.z;
      bool ok = gather_ok<Op::kEs>(g, dst, out, len, seq, n_src);
      for (uint32_t j = 0; ok && j < n_src; ++j) ok = gather_source_ok(g, d->src_off[j], len);
      if (ok) {
        const uint32_t bit = 1u << (seq & 31u);
        const uint32_t old = atomicOr(g.bitmap + (seq >> 5), bit);
        win = (old & bit) == 0;
      } else if (g.rejected != nullptr) {
        atomicAdd(g.rejected, 1u);
      }
    }
    const uint64_t winners = __ballot(win);
    const uint32_t pos = __popcll(winners & ((1ull << tid) - 1ull));
    const uint32_t count = __popcll(winners);
    if (win) {
      s.dst[pos] = dst;
      s.out[pos] = out;
      s.len[pos] = len;
      s.n_src[pos] = n_src;
      for (uint32_t j = 0; j < n_src; ++j) s.src[pos][j] = d->src_off[j];
    }
    if (tid == 0) s.count = count;
    const uint32_t vecs = (len >> 4) + ((len & 15u) != 0u ? 1u : 0u);  // no overflow for len up to 2^32 - 1
    const uint32_t units = win ? (vecs + kUnit - 1u) / kUnit : 0u;
    uint32_t incl = units;
#pragma unroll
    for (uint32_t dlt = 1; dlt < 64; dlt <<= 1) {
      const uint32_t below = __shfl_up(incl, dlt, 64);
      if (tid >= dlt) incl += below;
    }
    if (win) s.first[pos] = incl - units;
    if (tid == 63) s.first[count] = incl;
  }
  __syncthreads();

  const uint32_t count = s.count;
  const uint32_t total = s.first[count];
  const uint32_t wave = tid >> 6, lane = tid & 63u;
  for (uint32_t u = wave; u < total; u += NT / 64) {
    uint32_t w = 0;
    if (T > 1) {
      const bool mine = lane < count && s.first[lane] <= u && u < s.first[lane + 1];
      w = __ffsll(static_cast<unsigned long long>(__ballot(mine))) - 1;
    }
    w = __builtin_amdgcn_readfirstlane(w);
    const uint32_t v0 = (u - __builtin_amdgcn_readfirstlane(s.first[w])) * kUnit;
    gather_unit<U, ACC, Op>(g, wave_uniform(s.dst[w]), wave_uniform(s.out[w]), __builtin_amdgcn_readfirstlane(s.len[w]),
                            __builtin_amdgcn_readfirstlane(s.n_src[w]), s.src[w], v0, lane);
  }
}

// A call of few multi-source records: `parts` workgroups per record share its units (one compute
// unit reads a record's n + 1 streams far below its share of the memory system's rate: eight
// records of 128 KiB from seven senders take 25 us uncut).  The record's fate is decided once, by
// the first part to arrive (see claim_enter; a call of one part a record has no claim words); blockIdx.x = record * parts + part.  As in
// chunk_few_kernel every wavefront reads the record for itself and folds its first unit before the fate is
// known, so that the loads and the decision overlap (event pairs, seven sources, decided first -> folded first:
// 8 x 32 KiB 7.3 -> 6.7 us, 65 x 32 KiB 8.7 -> 8.0, 65 x 128 KiB 17.5 -> 16.1; three, 128 x 32 KiB 8.4 -> 7.6).
template <int NT, int U, class Op>
__global__ void __launch_bounds__(NT) chunk_gather_parts_kernel(const GatherArgs g) {
  constexpr uint32_t kUnit = 64u * U;
  constexpr uint32_t kWaves = NT / 64;
  constexpr int kBatch = 8 / U;
  __shared__ uint32_t s_win;
  const uint32_t tid = threadIdx.x, wave = tid >> 6, lane = tid & 63u;
  const uint32_t k = blockIdx.x / g.parts, part = blockIdx.x % g.parts;   // the launch has n_descs * parts workgroups
  const uccl_gather_desc* d = g.descs + k;
  const u32x4* p = reinterpret_cast<const u32x4*>(d);
  const u32x4 lo = p[0], hi = p[1];   // every lane reads the same 32 bytes
  const uint64_t so = d->src_off[lane & (UCCL_MAX_SOURCES - 1u)];   // lane j holds source j, named or not
  const uint64_t dst = wave_uniform(lo.x | (static_cast<uint64_t>(lo.y) << 32));
  const uint64_t out = wave_uniform(lo.z | (static_cast<uint64_t>(lo.w) << 32));
  const uint32_t len = __builtin_amdgcn_readfirstlane(hi.x);
  const uint32_t seq = __builtin_amdgcn_readfirstlane(hi.y);
  const uint32_t n_src = __builtin_amdgcn_readfirstlane(hi.z);
  const uint32_t vecs = (len >> 4) + ((len & 15u) != 0u ? 1u : 0u);
  const uint32_t total = (vecs + kUnit - 1u) / kUnit;
  const bool ok = gather_ok<Op::kEs>(g, dst, out, len, seq, n_src) && __all(lane >= n_src || gather_source_ok(g, so, len));
  const auto src = [so](uint32_t j) {
    const uint32_t a = __builtin_amdgcn_readlane(static_cast<uint32_t>(so), j), b = __builtin_amdgcn_readlane(static_cast<uint32_t>(so >> 32), j);
    return a | (static_cast<uint64_t>(b) << 32);
  };
  const uint32_t u0 = part * kWaves + wave;
  const bool have = ok && u0 < total;
  GatherUnit<U, Op> t;
  if (have) gather_fold<U, kBatch, Op>(g, t, dst, len, n_src, src, u0 * kUnit, lane);   // in bounds whatever the record's fate
  if (tid == 0) {
    uint32_t win = 0u;
    unsigned long long* const claim = g.claims + static_cast<size_t>(k) * UCCL_CLAIM_STRIDE;
    Claim entered = {true, 0ull};
    if (g.parts > 1u) entered = claim_enter<false>(claim, g.tag);   // the only part has nobody to agree with
    if (entered.decides) {
      if (ok) {
        const uint32_t bit = 1u << (seq & 31u);
        win = (atomicOr(g.bitmap + (seq >> 5), bit) & bit) == 0u ? 1u : 0u;
      } else if (g.rejected != nullptr) {
        atomicAdd(g.rejected, 1u);
      }
      if (g.parts > 1u) claim_publish<false>(claim, g.tag, win != 0u);
    } else if (ok && part * kWaves < total) {  // a part without units has nothing to wait for
      win = claim_await<false>(claim, entered.seen, g.tag, g.faults()) ? 1u : 0u;
    }
    s_win = win;
  }
  __syncthreads();
  if (s_win == 0u) return;   // uniform over the workgroup
  if (have) gather_store<U, kCached, Op>(g, t, dst, out, len, n_src, src, u0 * kUnit, lane);
  for (uint32_t u = u0 + kWaves * g.parts; u < total; u += kWaves * g.parts) {
    gather_fold<U, kBatch, Op>(g, t, dst, len, n_src, src, u * kUnit, lane);
    gather_store<U, kCached, Op>(g, t, dst, out, len, n_src, src, u * kUnit, lane);
  }
}

// Hundreds of records: decided 64 at a time, as in chunk_group_kernel; every wavefront folds its first unit meanwhile.  One
// vector a lane and all of up to eight sources in flight (two vectors, four sources: 600 x 8 KiB from seven 13.9 / 16.0 us).
template <class Op, bool PART_MAJOR>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_num_sgpr(80))) gather_group_kernel(const GatherArgs g) {
  constexpr int U = 1, kBatch = 8;
  constexpr uint32_t kUnit = 64u * U;
  constexpr uint32_t kWaves = 4;
  __shared__ DecideSlots s;
  __shared__ uint32_t s_win;
  const uint32_t tid = threadIdx.x, lane = tid & 63u;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const GroupPlace place = group_place<PART_MAJOR>(g);   // the launch has n_descs * parts workgroups
  const uint32_t k = place.k, part = place.part, in = place.in, base = place.base;
  const bool decides = UCCL_GROUP_LEADS && wave == 0u && place.first;
  unsigned long long* const line = g.claims + static_cast<size_t>(base / kGroup) * UCCL_CLAIM_STRIDE;
  unsigned long long was = 0ull;
  if (decides) {
    group_lead(line, g.tag);
    was = group_enter(line, g.tag, lane);
  }
  // every lane reads the workgroup's record; where the group is decided, lane i reads record i of the group
  const u32x4* p = reinterpret_cast<const u32x4*>(g.descs + (decides && base + lane < g.n_descs ? base + lane : k));
  u32x4 lo = p[0], hi = p[1];
  const uint64_t so = g.descs[k].src_off[lane & (UCCL_MAX_SOURCES - 1u)];   // lane j holds source j of record k, named or not
  const uint64_t dst = wave_uniform(lo.x | (static_cast<uint64_t>(lo.y) << 32));   // of lane 0: that is record k in either case
  const uint64_t out = wave_uniform(lo.z | (static_cast<uint64_t>(lo.w) << 32));
  const uint32_t len = __builtin_amdgcn_readfirstlane(hi.x);
  const uint32_t n_src = __builtin_amdgcn_readfirstlane(hi.z);
  const bool ok = gather_ok<Op::kEs>(g, dst, out, len, __builtin_amdgcn_readfirstlane(hi.y), n_src) &&
                  __all(lane >= n_src || gather_source_ok(g, so, len));
  const auto src = [so](uint32_t j) {
    const uint32_t a = __builtin_amdgcn_readlane(static_cast<uint32_t>(so), j), b = __builtin_amdgcn_readlane(static_cast<uint32_t>(so >> 32), j);
    return a | (static_cast<uint64_t>(b) << 32);
  };
  const uint32_t vecs = (len >> 4) + ((len & 15u) != 0u ? 1u : 0u);
  const uint32_t total = (vecs + kUnit - 1u) / kUnit;
  const uint32_t u0 = part * kWaves + wave;
  const bool have = ok && u0 < total;
  const bool part_has_units = ok && part * kWaves < total;   // uniform over the workgroup
  GatherUnit<U, Op> t;
  if (have && !decides) gather_fold<U, kBatch, Op>(g, t, dst, len, n_src, src, u0 * kUnit, lane);   // in bounds whatever the record's fate
  if (wave == 0u) {
    const bool win = group_outcome(
        line, g.tag, was, decides, part_has_units, in, lane, g.faults(),
        [&] {
          const u32x4* q = reinterpret_cast<const u32x4*>(g.descs + (base + lane < g.n_descs ? base + lane : k));
          lo = q[0];
          hi = q[1];
        },
        [&] {
          const bool is_record = base + lane < g.n_descs;
          bool good = is_record && gather_ok<Op::kEs>(g, lo.x | (static_cast<uint64_t>(lo.y) << 32), lo.z | (static_cast<uint64_t>(lo.w) << 32), hi.x, hi.y, hi.z);
          if (good) good = gather_sources_ok(g, g.descs + base + lane, hi.z, hi.x);
          if (is_record && !good && g.rejected != nullptr) atomicAdd(g.rejected, 1u);
          return __ballot(decide_wave(s, g.bitmap, good, hi.y, lane));
        });
    if (have && decides) gather_fold<U, kBatch, Op>(g, t, dst, len, n_src, src, u0 * kUnit, lane);
    if (lane == 0) s_win = win ? 1u : 0u;
  }
  if (!part_has_units) return;   // the whole workgroup
  __syncthreads();
  if (s_win == 0u) return;
  if (have) gather_store<U, kThrough, Op>(g, t, dst, out, len, n_src, src, u0 * kUnit, lane);
  for (uint32_t u = u0 + kWaves * g.parts; u < total; u += kWaves * g.parts) {
    gather_fold<U, kBatch, Op>(g, t, dst, len, n_src, src, u * kUnit, lane);
    gather_store<U, kThrough, Op>(g, t, dst, out, len, n_src, src, u * kUnit, lane);
  }
}

// A call of much payload: order and stream, as above.  What bounds it is the same, and a workgroup of 4 KiB
// of the destination keeps its n + 1 loads of one vector per lane in flight at once where the tile kernel
// walks 32 KiB and more (seven senders, fp32, 128 MiB in 128 KiB chunks: 256.5 us in the tile kernel, 208 here;
// 2 KiB parts 209, 8 KiB 211, two vectors per lane 217, without the contiguous runs 215, with six workgroups
// per compute unit 223, so the launch is not held back).
template <uint32_t kEs>
__global__ void __launch_bounds__(kOrderThreads) gather_order_kernel(const GatherArgs g, const OrderArgs t) {
  __shared__ DecideSlots s[kOrderThreads / 64];
  const uint32_t k = blockIdx.x * kOrderThreads + threadIdx.x;
  bool ok = false;
  uint32_t len = 0u, seq = 0u;
  if (k < g.n_descs) {
    const uccl_gather_desc* d = g.descs + k;
    const uint32_t n_src = d->n_src;
    len = d->len;
    seq = d->seq;
    ok = gather_ok<kEs>(g, d->dst_off, d->out_off, len, seq, n_src);
    if (ok) ok = gather_sources_ok(g, d, n_src, len);
    if (!ok && g.rejected != nullptr) atomicAdd(g.rejected, 1u);
  }
  if (decide_wave(s[threadIdx.x >> 6], g.bitmap, ok, seq, threadIdx.x & 63u)) order_put(t, g.n_descs, seq, k, len);
}

template <class Op>
__device__ __forceinline__ void ordered_gather_part(const GatherArgs& g, uint32_t k, uint32_t part) {
  constexpr uint32_t kUnit = 64u, kWaves = kOrderThreads / 64;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63u;
  const uccl_gather_desc* d = g.descs + k;   // the same address in every lane
  const uint32_t len = d->len;
  const uint32_t vecs = (len >> 4) + ((len & 15u) != 0u ? 1u : 0u);
  const uint32_t total = (vecs + kUnit - 1u) / kUnit;
  for (uint32_t u = part * kWaves + wave; u < total; u += g.parts * kWaves)
    gather_unit<1, kThrough, Op>(g, d->dst_off, d->out_off, len, d->n_src, d->src_off, u * kUnit, lane);
}

template <class Op>
__global__ void __launch_bounds__(kOrderThreads) gather_ordered_kernel(const GatherArgs g, const OrderArgs t) {
  const uint32_t b = order_position(g.n_descs * g.parts), entry = b / g.parts, part = (b + entry) % g.parts;
  const unsigned long long first = t.words[2u * static_cast<size_t>(entry)];
  const unsigned long long second = t.words[2u * static_cast<size_t>(entry) + 1u];
  if (order_has(t, first, part)) ordered_gather_part<Op>(g, order_record(first), part);
  if (order_has(t, second, part)) ordered_gather_part<Op>(g, order_record(second), part);
}

// ---- sender side: tensor buffer -> staged chunks + send records --------------------------------
//
// Section 2.1: the kernel copies from the tensor buffer to the transport buffer the NIC sends
// from; Section 3.1: the sender CPU names each chunk's address and sends a 32-bit control header
// with it.  A dense copy: chunk i of the range goes to slot i of the staging buffer, cut into
// 2 KiB units (64 lanes x 2 x 16 bytes), one unit per wavefront, 16 per workgroup.  The wavefront
// that takes a chunk's first unit also writes the chunk's send record.  The tensor is read with
// default policy (it is the accumulator, read again by the next step), staging is written
// non-temporally (the NIC reads it, the GPU does not).
struct SegmentArgs {
  char* stage;
  const char* tensor;
  uccl_send_desc* descs;
  uint64_t bytes;        // length of the range (tensor already points at its start)
  uint64_t slot_stride;
  uint64_t stage_off;    // of slot 0, for the records (stage already points there)
  uint64_t n_chunks;
  uint32_t chunk_bytes;
  uint32_t units_per_chunk;
  uint32_t conn_id, msg_id, first_csn;
};

__global__ void __launch_bounds__(1024) segment_kernel(const SegmentArgs g) {
  constexpr uint32_t kUnit = 128u;  // 16-byte vectors per unit
  const uint32_t lane = threadIdx.x & 63u;
  const uint64_t unit = static_cast<uint64_t>(blockIdx.x) * 16u + (threadIdx.x >> 6);
  const uint64_t i = unit / g.units_per_chunk;           // chunk
  const uint32_t u = static_cast<uint32_t>(unit % g.units_per_chunk);
  if (i >= g.n_chunks) return;                            // whole wavefronts leave; no barrier follows
  const uint64_t from = i * g.chunk_bytes;
  const uint64_t left = g.bytes - from;
  const uint32_t len = left < g.chunk_bytes ? static_cast<uint32_t>(left) : g.chunk_bytes;
  if (u == 0 && lane == 0 && g.descs != nullptr) {
    const uint64_t number = static_cast<uint64_t>(g.first_csn) + i;
    const uint32_t csn = static_cast<uint32_t>(number & 255u);
    const uint32_t msg = static_cast<uint32_t>((g.msg_id + (number >> 8)) & 127u);
    const uint32_t mark = (csn == 255u || i + 1 == g.n_chunks) ? 1u : 0u;
    uccl_send_desc d;
    d.stage_off = g.stage_off + i * g.slot_stride;
    d.len = len;
    d.header = csn | (mark << 8) | (msg << 9) | (g.conn_id << 16);
    g.descs[i] = d;
  }
  const uint32_t nvec = len >> 4;
  const uint32_t v0 = u * kUnit;
  const u32x4* sp = reinterpret_cast<const u32x4*>(g.tensor + from) + v0 + lane;
  u32x4* dp = reinterpret_cast<u32x4*>(g.stage + i * g.slot_stride) + v0 + lane;
  u32x4 v[2];
#pragma unroll
  for (int k = 0; k < 2; ++k)
    if (v0 + lane + k * 64 < nvec) v[k] = sp[k * 64];
#pragma unroll
  for (int k = 0; k < 2; ++k)
    if (v0 + lane + k * 64 < nvec) __builtin_nontemporal_store(v[k], dp + k * 64);
  const uint32_t rem = len & 15u;  // the last, partial vector: byte by byte, by the unit that holds it
  if (rem != 0u && nvec >= v0 && nvec < v0 + kUnit && lane < rem) {
    const uint64_t at = (static_cast<uint64_t>(nvec) << 4) + lane;
    g.stage[i * g.slot_stride + at] = g.tensor[from + at];
  }
}

__global__ void __launch_bounds__(256) fill_words_kernel(uint32_t* p, uint64_t n, uint32_t v) {
  for (uint64_t i = static_cast<uint64_t>(blockIdx.x) * 256 + threadIdx.x; i < n;
       i += static_cast<uint64_t>(gridDim.x) * 256)
    p[i] = v;
}

}  // namespace
