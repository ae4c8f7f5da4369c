// Receive-side chunk data path for multipath collectives, gfx950 (MI355X).
//
// One kernel does, per record of the arrival-ordered list the control path hands over
// (paper Section 3.1 "challenge of reassembly", Section 5): dedup by sequence number,
// place, combine with the tensor buffer (Section 2.1: "sum, max") or copy, write back,
// and forward to the outbound staging buffer.  The paper's own kernel first copies
// payloads into a transport buffer and then reduces; here the payload is read once,
// straight from its arrival slot, which gives the same result with 2x chunk size fewer
// bytes moved.
//
// Mapping onto the machine.  The work is a stream: at most one add per 4..8 bytes
// moved, so HBM bandwidth bounds it and no matrix core is involved.  A 1024-thread
// workgroup takes a tile of T consecutive records.  The lanes of its first wavefront each
// load one 32-byte record with two 128-bit loads, validate it, and test-and-set its bit
// with one device-scope atomic OR; the returned old word tells the lane whether it is the
// first arrival.  A wave ballot compacts the winners into LDS and a wave scan numbers
// their units (2 KiB; 1 KiB where a workgroup reduces a single record).  After one barrier
// the 16 wavefronts take units round-robin and stream them with 128-bit loads and stores:
// every thread issues all loads of a unit, then combines, then stores, and the workgroup
// retires.  Duplicates cost their record and one atomic, nothing else.  Two lanes holding
// the same seq each issue their own atomic, so the hardware serialises them and exactly one
// sees the bit clear.
//
// Calls of much payload are bound by how well the memory system takes their mix of reads and
// writes, which depends on the order of the accesses: they decide all sequence numbers in a small
// launch of its own and stream the winners in destination order in a second one.
//
// Calls of hundreds of records take a record, or a part of one, a workgroup and load its payload at once, while one
// wavefront of every 64 records decides them for the others.
//
// Calls of few records (Appendix C.4: small messages are where fixed costs show) take another
// kernel, which shortens the chain of latencies instead: one record per workgroup, payload
// loads issued before the sequence number is decided, and, when the records alone would leave
// most compute units idle, each record cut into parts over several workgroups that agree on
// its fate through claim words in scratch memory (uccl_data_kernels.hpp).  The sender side
// (tensor range -> staged chunks + send records) and the feedback kernels (acknowledgement
// report, per-message status) are dense, small kernels of their own.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include <atomic>
#include <mutex>
#include <new>
#include <tuple>
#include <utility>

#include "uccl_chunk.h"

#include "uccl_elements.hpp"
#include "uccl_data_kernels.hpp"
#include "uccl_feedback_kernels.hpp"

// Scratch memory: arrays inside the library's code object, so that no call allocates.  Every GPU the
// library runs on holds its own copy, zero at first, at its own address until the process ends.  In host code
// the names only stand for the symbols: the device addresses are looked up per device (device_array).

// Claim words for uccl_chunk_apply_noalloc (see claim_enter): a record's two on a
// 128-byte line of their own, UCCL_NOALLOC_MAX_DESCS of them, then the word that counts parts that
// gave up waiting: 256.25 KiB.
static __device__ __align__(256) unsigned long long scratch[UCCL_NOALLOC_MAX_DESCS * UCCL_CLAIM_STRIDE + 32];

// The regions that streams own (see claim_region), large ones first, then the same counter: 36.5 MiB.
constexpr uint32_t kRegionRecords = 2048;  // most records a split call can have
constexpr uint32_t kRegionWords = kRegionRecords * UCCL_CLAIM_STRIDE;
constexpr uint32_t kGroupRegionWords = 48 * UCCL_CLAIM_STRIDE;   // calls of hundreds of records: a line for 64 of them
enum RegionUse : uint32_t { kCutCalls, kOtherCalls, kThreads, kGroupCalls, kGroupThreads, kRegionUses };
constexpr uint32_t kStreamRegions = 64, kThreadRegions = 16;   // streams with regions, for each use; threads
constexpr uint32_t kLargeRegions = 2 * kStreamRegions + kThreadRegions, kRegions = kLargeRegions + kStreamRegions + kThreadRegions;
constexpr size_t kAllRegionWords = static_cast<size_t>(kLargeRegions) * kRegionWords + static_cast<size_t>(kRegions - kLargeRegions) * kGroupRegionWords;
static __device__ __align__(256) unsigned long long regions[kAllRegionWords + 32];

namespace {

// ---- host side ----------------------------------------------------------------------

thread_local char t_detail[256] = "";
thread_local hipEvent_t t_start = nullptr, t_stop = nullptr;  // one-shot, see uccl_time_next_launch

int launch_failed(hipError_t e) {
  snprintf(t_detail, sizeof(t_detail), "%s: %s", hipGetErrorName(e), hipGetErrorString(e));
  return UCCL_ELAUNCH;
}

// Launch through the calls that RETURN the launch status (the <<<>>> form leaves it in the
// thread's last-error slot, where an earlier, unrelated error could be mistaken for ours and
// reading it would clear the caller's).  The one-shot timing events, if any, are attached to
// this very dispatch.
template <class... Params, size_t... I>
hipError_t launch_raw(void (*kernel)(Params...), dim3 grid, dim3 block, uint32_t lds, hipStream_t s,
                      std::tuple<Params...>& params, std::index_sequence<I...>) {
  void* ptrs[] = {static_cast<void*>(&std::get<I>(params))...};
  hipEvent_t t0 = t_start, t1 = t_stop;
  t_start = t_stop = nullptr;
  if (t0 != nullptr || t1 != nullptr)
    return hipExtLaunchKernel(reinterpret_cast<const void*>(kernel), grid, block, ptrs, lds, s, t0, t1, 0);
  return hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, block, ptrs, lds, s);
}

// `lds`: dynamic LDS per workgroup.
template <class... Params, class... KernelArgs>
int launch_kernel_lds(void (*kernel)(Params...), uint32_t tiles, uint32_t threads, uint32_t lds, hipStream_t s, KernelArgs... a) {
  static_assert(sizeof...(Params) == sizeof...(KernelArgs), "one argument per kernel parameter");
  std::tuple<Params...> params(static_cast<Params>(a)...);  // objects of the kernel's own parameter types
  const hipError_t e = launch_raw(kernel, dim3(tiles), dim3(threads), lds, s, params, std::index_sequence_for<Params...>{});
  return e == hipSuccess ? UCCL_OK : launch_failed(e);
}

template <class... Params, class... KernelArgs>
int launch_kernel(void (*kernel)(Params...), uint32_t tiles, uint32_t threads, hipStream_t s, KernelArgs... a) {
  return launch_kernel_lds(kernel, tiles, threads, 0u, s, a...);
}

uint32_t tiles_for(uint32_t n_descs, uint32_t tile) {
  return static_cast<uint32_t>((static_cast<uint64_t>(n_descs) + tile - 1) / tile);
}

// ---- scratch regions ----------------------------------------------------------------------------
//
// Scratch memory of the split launch (see claim_enter): one 64-bit word per record of the call,
// on a 128-byte line of its own.  Ordered calls keep their table in the same words
// (chunk_order_kernel), the acknowledgement report its segments' counts (ack_segments_kernel); every
// word carries the tag of the call that wrote it in bits 16 and up, whatever the call, so each kind
// finds the others' words stale.  Every device has kRegions regions for
// kRegionRecords records each, one per stream handle that has issued such a call: one for its cut calls and another
// for everything else, so that streams which only ask for reports, say, leave the cut calls theirs (these gain
// most); and small ones for calls of hundreds of records, which any stream may have.  Calls on
// one stream run in order, so they can share a region; calls on different streams may overlap, so
// they never do.  A call whose stream finds no free region, or that is being captured into a graph
// (a replay would carry the captured tag again, and could overlap with anything), is launched in the
// form that needs none.
//
// Tags come from one process-wide counter.  A call draws its tag and enqueues its launches while holding its
// region's launch lock: claim words need tags that grow in the order in which the
// calls of a region run, and the launches of two ordered calls on one stream must not come between each other, also
// when several host threads issue calls on that stream.  A launch may wait for room in its stream's queue; calls on
// other streams do not wait with it.
constexpr int kMaxDevices = 64;

struct RegionOwners {
  std::mutex lock;                       // guards the table's growth
  std::atomic<uint32_t> n{0};
  std::atomic<uintptr_t> key[kStreamRegions];
};
struct ClaimPool {
  RegionOwners owners[kRegionUses];
  std::mutex launch_lock[kRegions];      // a region's: held from drawing a tag until its launches are enqueued
};
ClaimPool g_pools[kMaxDevices];
std::atomic<unsigned long long> g_next_tag{2};  // tags are unique across streams, devices and threads; 1 is for captured calls

// One of the arrays above, by device: its address once it has been looked up with that device current.
struct DeviceArray {
  std::atomic<unsigned long long*> at[kMaxDevices];
};
DeviceArray g_scratch, g_regions;

// The look-up loads the library's code object if nothing has yet; the thread's capture checks are relaxed
// meanwhile, for another stream of the program may be under capture, which that does not concern.
int device_array(DeviceArray& array, const void* symbol, int dev, unsigned long long** out) {
  unsigned long long* p = array.at[dev].load(std::memory_order_acquire);
  if (p == nullptr) {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    const bool relaxed = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
    void* at = nullptr;
    const hipError_t e = hipGetSymbolAddress(&at, symbol);
    if (relaxed) (void)hipThreadExchangeStreamCaptureMode(&mode);
    if (e != hipSuccess) return launch_failed(e);
    if (at == nullptr) return UCCL_ELAUNCH;
    p = static_cast<unsigned long long*>(at);
    array.at[dev].store(p, std::memory_order_release);   // whoever else looks it up finds the same
  }
  *out = p;
  return UCCL_OK;
}

int current_device(int* dev) {
  const hipError_t e = hipGetDevice(dev);
  if (e != hipSuccess) return launch_failed(e);
  return *dev < 0 || *dev >= kMaxDevices ? UCCL_EINVAL : UCCL_OK;
}

uint32_t* region_faults(unsigned long long* base) {
  return reinterpret_cast<uint32_t*>(base + kAllRegionWords);
}

// Whose region it is: 0 marks a free entry, the null stream is 1.  hipStreamPerThread is one handle for a stream of each
// thread, and those may overlap.  A thread goes by a number that no other thread ever has: its work may go on after it
// has ended (the runtime does not wait there, as it does in hipStreamDestroy), when the next thread may have its
// addresses.  Regions are not given back, so threads have a few of their own, for any use, and a program that keeps starting them takes no
// stream's away.
uintptr_t region_key(hipStream_t stream) {
  if (stream != hipStreamPerThread) return 1 + reinterpret_cast<uintptr_t>(stream);
  static std::atomic<uintptr_t> threads{0};
  static thread_local const uintptr_t mine = threads.fetch_add(1, std::memory_order_relaxed);
  return ~mine;   // no address
}

// A region of `stream` on the current device; no words: there is none to be had, or the stream is being captured.
struct Region {
  unsigned long long* words = nullptr;
  uint32_t* faults = nullptr;
  std::mutex* launch_lock = nullptr;
};

Region claim_region(hipStream_t stream, RegionUse use) {
  Region r;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) { (void)hipGetLastError(); return r; }
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(stream, &cap) != hipSuccess) { (void)hipGetLastError(); return r; }
  if (cap != hipStreamCaptureStatusNone) return r;
  unsigned long long* base = nullptr;
  if (device_array(g_regions, HIP_SYMBOL(regions), dev, &base) != UCCL_OK) { (void)hipGetLastError(); return r; }
  if (stream == hipStreamPerThread) use = use == kGroupCalls ? kGroupThreads : kThreads;
  constexpr uint32_t kFirst[kRegionUses] = {0, kStreamRegions, 2 * kStreamRegions, kLargeRegions, kLargeRegions + kStreamRegions};
  RegionOwners& o = g_pools[dev].owners[use];
  const uintptr_t key = region_key(stream);
  uint32_t n = o.n.load(std::memory_order_acquire), at = 0;
  while (at < n && o.key[at].load(std::memory_order_relaxed) != key) ++at;
  if (at == n) {
    std::lock_guard<std::mutex> hold(o.lock);
    n = o.n.load(std::memory_order_acquire);
    while (at < n && o.key[at].load(std::memory_order_relaxed) != key) ++at;   // only the new entries: old ones stay
    if (at == n) {
      if (n == (use == kThreads || use == kGroupThreads ? kThreadRegions : kStreamRegions)) return r;
      o.key[n].store(key, std::memory_order_relaxed);
      o.n.store(n + 1, std::memory_order_release);
    }
  }
  const uint32_t index = kFirst[use] + at;
  r.words = index < kLargeRegions ? base + static_cast<size_t>(index) * kRegionWords
                                  : base + static_cast<size_t>(kLargeRegions) * kRegionWords + static_cast<size_t>(index - kLargeRegions) * kGroupRegionWords;
  r.faults = region_faults(base);
  r.launch_lock = &g_pools[dev].launch_lock[index];
  return r;
}

// Per-call tuning (uccl_launch_opts); zero = let the library decide.  static_claims: the call
// uses these claim words and no region.
struct Tuning {
  uint32_t chunk_bytes;
  uint32_t parts;
  unsigned long long* static_claims = nullptr;
  bool one_launch = false;  // the call may be offered again after an error: all of it is enqueued, or nothing
};

template <int T, int U, class Op, Through H = kNoThrough>
int launch_flat(const Args& a, hipStream_t s) {
  uint32_t tiles = tiles_for(a.n_descs, T);
  if (UCCL_XCD_CONTIGUOUS) tiles = (tiles + 7u) / 8u * 8u;   // whole eighths; tiles past the records find none
  return launch_kernel(chunk_flat_kernel<UCCL_FLAT_THREADS, T, U, Op, H>, tiles, UCCL_FLAT_THREADS, s, a);
}

template <class Op, Through H>
int launch_tiles(const Args& a, hipStream_t s, uint32_t tile) {
  if (tile >= 8) return launch_flat<8, UCCL_FLAT_UNROLL, Op, H>(a, s);
  if (tile >= 4) return launch_flat<4, UCCL_FLAT_UNROLL, Op, H>(a, s);
  return launch_flat<2, UCCL_FLAT_UNROLL, Op, H>(a, s);
}

// Records per workgroup: enough that a tile holds about 32 KiB of payload per stream when the
// chunk size is known, otherwise grown with the record count.
uint32_t flat_tile(uint32_t n_descs, uint32_t chunk_bytes) {
  uint32_t t;
  if (chunk_bytes) {
    t = (32768u + chunk_bytes - 1) / chunk_bytes;
  } else {
    // Unknown chunk size: a tile too large for big chunks costs a few percent, a tile too
    // small for 4 KiB chunks costs a factor of two, so grow the tile once the record count
    // leaves enough workgroups either way.
    t = n_descs < 8192u ? 1u : n_descs < 32768u ? 4u : n_descs < 131072u ? 8u : 16u;
  }
  return t < 1u ? 1u : t > 32u ? 32u : t;
}

// Calls of fewer single-record tiles than this are launched with chunk_few_kernel (measured with
// 32 / 64 / 128 KiB chunks and no duplicates: 512 records 12-20 % faster than chunk_flat_kernel,
// 1024 records 1-9 %, 2048 records 1-3 %; a duplicate costs chunk_few_kernel its payload reads, so
// large calls, where the difference has gone, stay with chunk_flat_kernel).
#ifndef UCCL_FEW_RECORDS
#define UCCL_FEW_RECORDS 2048
#endif
constexpr uint32_t kFewRecords = UCCL_FEW_RECORDS;
// Payload bytes per stream that one part's wavefronts take in their first, eagerly loaded trip.
constexpr uint32_t kPartBytes = UCCL_PART_THREADS * UCCL_PART_UNROLL * 16u;

// Workgroups per record for a call of few single-record tiles.  One compute unit moves its record's
// 3-4 streams at a small fraction of the memory system's rate, so while the records alone leave
// compute units idle a record is spread over several of them.  Measured (kernel time, fp32 SUM with
// forward, records x chunk size: uncut -> cut): 57 x 64 KiB 6.4 -> 5.2 us in 8 parts; 256 x 64 KiB
// 14.6 -> 12.4 us in 8; 128 x 128 KiB 17.4 -> 12.3 us in 16; 256 x 128 KiB 25.8 -> 24.1 us in 8;
// 32 x 32 KiB 4.4 -> 4.1 us in 8; but 128 x 32 KiB 5.6 -> 5.9 us in 4 and 512 x 64 KiB 24.7 ->
// 25.4 us in 8.  Hence: chunks above 32 KiB are cut into parts of about 8 KiB (at most 16) while
// the call holds at most 16 MiB of payload and the launch stays within 2048 workgroups; chunks of
// up to 32 KiB only in calls of at most 32 records; with the chunk size unknown, by record count
// alone.  Parts that find no unit in a shorter record leave at once.
uint32_t auto_parts(uint32_t n_descs, uint32_t chunk_bytes) {
  if (chunk_bytes == 0u) return n_descs <= 64u ? 8u : n_descs <= 128u ? 4u : 1u;
  if (chunk_bytes <= 32768u) return n_descs <= 32u && chunk_bytes > kPartBytes ? 8u : 1u;
  if (static_cast<uint64_t>(n_descs) * chunk_bytes > (16ull << 20)) return 1u;
  uint32_t parts = 16u;
  while (parts > 1u && parts * kPartBytes > chunk_bytes) parts /= 2u;   // about kPartBytes per part
  while (parts > 1u && n_descs * parts > 2048u) parts /= 2u;
  return parts;
}

// Calls of few small chunks (a message of a few dozen 4 KiB packets) take chunk_few_kernel with one
// small workgroup per record instead of a tile of records per large workgroup: the call is far too
// small to fill the machine either way, and the shorter chain of latencies wins (kernel time, fp32
// SUM with forward, 57 records: 4 KiB 4.7 -> 3.1 us, 8 KiB 5.3 -> 3.3 us, 16 KiB 5.6 -> 3.7 us; 128
// records 15-30 % faster; 512 records of 4 or 8 KiB 15-45 % slower, hence the limit).  Chunks above
// 8 KiB fill a workgroup and keep an edge for much longer (16 KiB: 1024 records 15 % faster, 4096
// records 10 %, 8192 records 1 %); one 16-byte vector per lane of a 1024-thread workgroup covers a
// 16 KiB chunk in one trip and is 2-6 % faster than two vectors per lane of a 512-thread one
// (all-to-all of 3 600 records 21.2 against 21.6 us, 1 024 reduced records 14.3 against 15.3 us).
#ifndef UCCL_SMALL_CALL_RECORDS
#define UCCL_SMALL_CALL_RECORDS 128
#endif
#ifndef UCCL_HALF_TILE_RECORDS
#define UCCL_HALF_TILE_RECORDS 8192
#endif
constexpr uint32_t kSmallCallRecords = UCCL_SMALL_CALL_RECORDS;
constexpr uint32_t kHalfTileRecords = UCCL_HALF_TILE_RECORDS;

// Which launch a call gets: decided here, in one place, from the record count and the tuning alone
// (pure host arithmetic; uccl_launch_plan reports it).  `parts` > 1 is a wish: it needs claim words,
// and a call that finds none (no free region, stream being captured) takes the uncut route instead.
enum Route : uint32_t {
  kRouteTile,       // chunk_flat_kernel, `tile` >= 2 records per workgroup
  kRouteOne,        // chunk_flat_kernel, one record per workgroup
  kRouteFew,        // chunk_few_kernel, one UCCL_FEW_THREADS workgroup per record (calls of < kFewRecords large records)
  kRouteParts,      // chunk_few_kernel, `parts` workgroups of UCCL_PART_THREADS per record
  kRouteHalf,       // chunk_few_kernel<1024, 1>: chunks of 8-16 KiB, one workgroup per record
  kRouteSmall1,     // chunk_few_kernel<256, 1>: at most kSmallCallRecords chunks of up to 4 KiB
  kRouteSmall2,     // chunk_few_kernel<256, 2>: the same, chunks of up to 8 KiB
};
struct Plan {
  Route route;
  uint32_t tile, parts, threads, unroll;
};

// Calls of much payload decide all sequence numbers first and stream the winners in destination order
// (chunk_order_kernel, chunk_ordered_kernel).  The order launch takes 4.6 us behind another kernel (6.0 - 6.4 in
// the measures below, which a threshold owes 1.5 us), the order gains more the
// more streams the call has and the larger its chunks are.  Measured on the two kinds of board of this
// machine (the second mixes reads and writes better), us, this form / the other; ring steps, bf16, the
// reduce phase ordered alone: 56 MiB of payload in 32 KiB chunks 73.0 / 70.2 (second kind); 112 MiB 134 / 139
// and 132 / 135; 168 MiB in 16 KiB chunks 194 / 204 and 195 / 191, in 128 KiB chunks 198 / 225 and 194 / 203;
// 896 MiB in 128 KiB chunks 563 / 689; 224 MiB in 9 KB chunks 279 / 265 (second kind).  The copy phase too, against
// the reduce phase alone: 112 MiB in 32 KiB chunks 136 / 134 and 134 / 132, 168 MiB in 128 KiB chunks 191 / 198
// and 191 / 194, 240 MiB in 32 KiB chunks 268 / 270, 224 MiB in 20 KB chunks 258 / 261 and 252 / 260.
// Several sources per record (how many, the host does not know), 128 KiB chunks: 48 MiB of destination from one
// source 35.3 / 32.4, from seven 82.7 / 90.0; 96 MiB 64.1 / 65.7 and 164 / 197; in 32 KiB chunks 66.0 / 69.8 and 172 / 190.
//
// With the chunk size unknown the same form is taken for another reason too.  A workgroup per record decides
// its sequence number with an atomic of its own, atomics of neighbouring records meet on one 128-byte line of
// the bitmap, and such atomics are served one after the other, about 6.5 ns each: 5000 records take 30 us whatever
// their size, while the order kernel's wavefronts issue 64 at a time.  Four parts an entry suit records of any
// size (ring steps over three sets of buffers, us, this form / one workgroup per record: 28 MiB in 4 KiB chunks 56 / 91, 64 MiB
// in 9 KB 84 / 108, 256 MiB in 32 KiB 275 / 291, 400 MiB in 64 KiB 515 / 528; all-to-all, chunks of 8 KiB 29 / 35, of 16 KiB 35.4 / 33.0, of
// 64 KiB 117 / 120).  Entries by arrival instead would lose no order where windows of sequence numbers are partly used (64 of 256:
// 5000 of 4 KiB 28 by sequence number, 23 by arrival, 32 other form; of 16 KiB 64, 48, 55), but all of it elsewhere (256 MiB in 32 KiB 294).
// Where the alternative is tiles of four records (8192 and more), whose atomics are few, the other form is taken: small
// records lose too much to workgroups without work (16 383 of 64 B 44 / 31, 60 MiB in 4 KiB 91 / 85; windows partly used 44 / 25),
// for what 16 - 24 KiB chunks would gain (256 MiB 281 / 308).
//
// A record shorter than stated leaves workgroups without work, at about 0.43 ns each, which the host cannot know: 8000
// records of 4 KiB stated as 128 KiB 144 / 53, as 32 KiB 47 / 53.  So no record has more than kOrderMaxParts of them: 8000 of
// 4 KiB stated as 1 MiB 144 instead of 260 with 64, for 7 - 10 % on chunks that are that large (3072 of 256 KiB 534 / 641, 496 with
// 64 parts).
//
// Records in pinned host memory are read across the bus once by the order kernel and again by every part of theirs;
// the other form reads them once (same measures, records in pinned memory: 7856 of 32 KiB 160 / 149, copies 123 / 105; 16 383
// of 4 KiB of unknown size 77 / 54).  Asking the runtime where they are takes 0.1 us of the host's time.
//
// `launches`: of each kernel (the table holds kOrderRecords entries; more records are
// taken in equal shares, each of which has to be worth it), 0 = not this form.  Needs a region;
// a stated number of parts asks for the other form.  The batcher's hand-overs stay with the other form: a hand-over
// that fails is offered again, so it must not leave sequence numbers decided whose payload has not moved, and its
// chunk size is the largest length in it, which may be one record's.
constexpr uint32_t kOrderRecords = 0x3FFFu;
static_assert(2u * kOrderRecords <= kRegionWords, "two words each; a table entry has 14 bits for the record");
constexpr uint32_t kOrderChunk = 16u << 10;
constexpr uint64_t kOrderBytes = 96ull << 20;
constexpr uint32_t kOrderCopyChunk = 64u << 10;        // copies: chunks of this size from kOrderBytes on,
constexpr uint64_t kOrderCopyBytes = 192ull << 20;     // smaller ones from here on
constexpr uint32_t kOrderUnknownRecords = 3072;        // chunk size unknown: from this many records
constexpr uint32_t kOrderUnknownTiles = 8192;          // to less than this many: tiles from here on (flat_tile)
constexpr uint32_t kOrderUnknownParts = 4;
constexpr uint32_t kMaxLaunchThreads = 0xFFFFFFFFu;    // HIP counts a launch's threads in 32 bits
constexpr uint32_t kOrderMaxParts = 32;   // longer records are walked

bool in_device_memory(const void* p) {
  hipPointerAttribute_t a;
  if (hipPointerGetAttributes(&a, p) == hipSuccess) return a.type == hipMemoryTypeDevice;
  (void)hipGetLastError();
  return false;
}

struct OrderPlan {
  uint32_t launches, parts;
};
constexpr OrderPlan kNotOrdered = {0u, 1u};

OrderPlan plan_ordered(uint32_t n_descs, const Tuning& tune, bool reads_acc, bool gather) {
  if (tune.parts == 0u && tune.chunk_bytes == 0u && !gather)
    return n_descs >= kOrderUnknownRecords && n_descs < kOrderUnknownTiles ? OrderPlan{1u, kOrderUnknownParts} : kNotOrdered;
  if (tune.parts != 0u || tune.chunk_bytes < kOrderChunk || n_descs == 0u) return kNotOrdered;
  // A count that is too large for the form of one launch is refused there, before anything is enqueued: a count that
  // is none (-1) must not become a quarter of a million launches.
  if (tiles_for(n_descs, flat_tile(n_descs, tune.chunk_bytes)) > kMaxLaunchThreads / UCCL_FLAT_THREADS) return kNotOrdered;
  const uint32_t launches = (n_descs - 1u) / kOrderRecords + 1u;
  const uint64_t least = reads_acc || tune.chunk_bytes >= kOrderCopyChunk ? kOrderBytes : kOrderCopyBytes;
  if (static_cast<uint64_t>(n_descs / launches) * tune.chunk_bytes < least) return kNotOrdered;
  const uint32_t parts = (tune.chunk_bytes - 1u) / kOrderPartBytes + 1u;
  return {launches, parts < kOrderMaxParts ? parts : kOrderMaxParts};
}

Plan plan_apply(uint32_t n_descs, const Tuning& tune, bool reads_acc) {
  const uint32_t t = flat_tile(n_descs, tune.chunk_bytes);
  if (t >= 2 && tune.chunk_bytes > 8192u && n_descs < kHalfTileRecords) return {kRouteHalf, 1u, 1u, 1024u, 1u};
  if (t >= 2 && tune.chunk_bytes != 0u && n_descs <= kSmallCallRecords) {
    // workgroup sized to the chunk: one trip of 16 bytes x unroll per lane covers it
    if (tune.chunk_bytes <= 4096u) return {kRouteSmall1, 1u, 1u, 256u, 1u};
    return {kRouteSmall2, 1u, 1u, 256u, 2u};
  }
  if (t >= 2) return {kRouteTile, t >= 32 ? 32u : t >= 16 ? 16u : t >= 8 ? 8u : t >= 4 ? 4u : 2u, 1u, UCCL_FLAT_THREADS, UCCL_FLAT_UNROLL};
  const uint32_t parts = tune.parts ? tune.parts : (n_descs < kFewRecords ? auto_parts(n_descs, tune.chunk_bytes) : 1u);
  if (parts > 1u && n_descs <= kRegionRecords) return {kRouteParts, 1u, parts, UCCL_PART_THREADS, UCCL_PART_UNROLL};
  if (n_descs < kFewRecords) return {kRouteFew, 1u, 1u, UCCL_FEW_THREADS, UCCL_FEW_UNROLL};
  // One record per workgroup.  Kernels that read the accumulator take 1 KiB units here (a wavefront
  // makes two trips through a 32 KiB chunk, eight through a 128 KiB one, its stores of one trip
  // between the loads of two): measured 0.7 % faster on 32 KiB chunks and 1.9 % on 128 KiB ones
  // than 2 KiB units; copies are 5 % slower that way and keep 2 KiB units.
  const uint32_t unroll = reads_acc ? UCCL_FLAT1_REDUCE_UNROLL : UCCL_FLAT_UNROLL;
  return {kRouteOne, 1u, 1u, UCCL_FLAT_THREADS, unroll};
}

// Calls of hundreds of records are decided 64 records at a time (chunk_group_kernel).  This form needs a region and records
// in device memory (each workgroup reads its record four times), a count known to the host (the indirect call's
// capacity may be mostly empty) and no stated number of parts.
//
// Workgroups and where the lines lie (ring steps of reduce and copy phase with reset over three sets of buffers, 130 - 2900
// records, 4 - 128 KiB, us, the form before / this one; all-to-all alike).  Four wavefronts a workgroup, a trip of one, two or
// four vectors a lane that covers the chunk, longer chunks 16 KiB a workgroup:
//   to 8 KiB: 130 records 11.0 / 11.2, 200 11.7 / 11.0, 900 x 4 KiB 16.8 / 14.6, 1800 x 6 KB 29.8 / 22.5, 2900 x 8 KiB 42.0 / 38.9,
//             5120 x 4 KiB 40 / 43
//   to 16 KiB (before: a workgroup of 1024 a record): 260 15.1 / 15.2, 330 x 16 KiB 16.2 / 15.8, 900 x 9 KB 27.3 / 18.6; 5120 x 16 KiB 101 / 105
//   to 32 KiB: 200 16.6 / 16.7, 260 21.6 / 18.8, 640 36.0 / 32.5; 1280 54.8 / 57.3
//   above, from where a call is no longer cut into parts: 260 x 64 KiB 35.3 / 26.9, 330 38.1 / 33.4; 1280 98.5 / 103
// With the size unknown, two to four parts of 16 KiB, all records' first ones first (group_place), so that a call in which some
// records are long does not wait for one workgroup to walk each of them: as many parts as cost records of 4 KiB
// next to nothing.  Measured, us a pass of reset and call, a workgroup of 1024 that decides for itself / one part here / this,
// SUM with forward (COPY):
//   four parts, to 640 records (one part: of 512 threads): 192 x 64 KiB 13.1 / 13.8 / 11.3 (8.9 / 9.3 / 8.0), 256 x 64 KiB 15.5 / 16.7 / 13.3, 480 x 4 KiB 9.8 / 6.9 / 6.8, 480 x 128 KiB
//     43.1 / 42.8 / 43.7; 400 records of 4 - 256 KiB, spread over the logarithm, 42.7 / 43.2 / 27.6, of 64 B - 1 MiB 125 / 122 / 57
//   three, to 1500: 900 x 64 B, 4, 64 KiB 10.4 / 6.2 / 7.0, 11.5 / 7.1 / 7.8, 41.8 / 41.8 / 41.0; 900 of 4 - 256 KiB 54.4 / 67.8 / 51.5 (46.2 / 58.8 / 43.0; two parts
//     57.0, four 46.8); 1280 x 4 KiB 13.4 / 8.4 / 8.6
//   two: 2000 x 4, 16, 64 KiB 16.3 / 10.7 / 10.4, 26.0 / 25.5 / 26.4, 105 / 103 / 103; 2000 of 4 - 256 KiB 118 / 138 / 121 (three parts 116, but 12.0 for the 4 KiB
//     ones); 3000 x 4 KiB 22.6 / 14.0 / 14.8, of 64 B - 1 MiB 359 / 375 / 335
// Where they lose to the forms before: a call of duplicates only, whose payload is read for nothing (2900 x 4 KiB 7.2 / 8.4); sequence numbers of which no two share a bitmap word (2900 x 4 KiB 13.2 / 13.8); few records much shorter than stated
// (192 x 2 KiB stated as 8 KiB 5.3 / 5.8, as 200 KiB 6.2 / 7.0).
constexpr uint32_t kGroupThreads = 256;
struct GroupPlan {
  uint32_t unroll, parts;   // vectors a lane and trip (0 = not this form), workgroups a record
};
constexpr GroupPlan kNotGrouped = {0u, 0u};
constexpr uint32_t kGroupFewest = 192u;
constexpr uint32_t kGroupMost = 3000u;
constexpr uint32_t kGatherSmallRecords = 288u;  // folds of small chunks: cut into parts to this many (gather_parts)
constexpr uint64_t kGroupBytes = 40ull << 20;   // of payload, in chunks above 8 KiB
static_assert((kGroupMost + kGroup - 1) / kGroup * UCCL_CLAIM_STRIDE <= kGroupRegionWords, "a line a group");

GroupPlan plan_group(uint32_t n_descs, const Tuning& tune) {
  if (tune.parts != 0u || n_descs < kGroupFewest || n_descs > kGroupMost) return kNotGrouped;
  const uint32_t chunk = tune.chunk_bytes;
  if (chunk == 0u) return {4u, n_descs <= 640u ? 4u : n_descs <= 1500u ? 3u : 2u};
  if (chunk <= 4096u) return {1u, 1u};
  if (chunk <= 8192u) return {2u, 1u};
  const uint64_t bytes = static_cast<uint64_t>(n_descs) * chunk;
  const GroupPlan p = {4u, (chunk - 1u) / 16384u + 1u};
  if (chunk <= 16384u) return n_descs >= 320u && bytes <= kGroupBytes ? p : kNotGrouped;
  if (chunk <= 32768u) return n_descs >= 256u && bytes <= (24ull << 20) ? p : kNotGrouped;
  return bytes > (16ull << 20) && bytes <= kGroupBytes ? p : kNotGrouped;
}

// The same for folds (gather_group_kernel); workgroups per record, 0 = not this form.  How many sources a record has, the
// host does not know: the lines lie where one source loses nothing to speak of.  The forms before come in rounds of 256 workgroups of
// 1024, one a compute unit (they take 66 registers and more), and a round costs the same however full it is, so what this form gains depends on how
// full the last of those is.  Above 32 KiB a workgroup of theirs takes a record: taken where their first round is to 160 / 256 full, or their second to 104 / 256
// (360 records).  4 - 8 KiB, tiles of four: not where one round is 160 / 256 full and more.
// Measured (fold with reset over three sets of buffers, sources 1, 2 or 3, 7, us or ratio, before / now):
//   small chunks, from where they are no longer cut into parts: 300 x 4, 8 KiB 1.03 1.02 1.57, 1.04 1.11 1.44; 1500 1.09 1.13 1.09, 1.22 1.17 1.15; 2800 1.05 1.04 1.10,
//       1.13 1.16 1.14.  Two workgroups a chunk of 8 KiB while the chip holds them all (600 8.2 9.3 12.9 us, one 9.2 10.2 13.2; 1200 13.6 16.2 22.3, one
//       11.6 14.4 20.5).  Not 640 - 1024 in chunks above 4 KiB, one tile of four each compute unit: 760 and 830 x 6 KB 0.97 0.97 0.94, 0.90 0.92 0.97
//   9 KB 1000 0.90 0.88 0.93; 16 KiB 470 0.94 0.97 1.05, 700 1.18 1.14 1.20, 1240 1.09 1.11 1.16, 2400 0.95 1.05 1.04
//   larger ones, not cut into parts above 16 MiB: 32 KiB 530 1.03 1.00 1.22, 850 1.00 1.02 1.17, 1200 0.97 1.06 1.07; 132 and 150 x 128 KiB 1.03 1.01 1.21, 1.00 1.01 1.18,
//       180 x 96 KiB 0.92 0.97 1.13, 200 x 128 KiB 0.93 1.01 1.12; 262, 300 x 128 KiB 1.14 1.20 1.38, 1.08 1.13 1.28, 350 x 48 KiB 1.07 1.08 1.12, 400 x 96 KiB 0.92 1.00 1.11
//   fewer and larger: no less worth it (f32 SUM of seven sources, f16 MAX of one): 1 x 48 MiB 8520 / 84, 3550 / 36, 16 x 2 MiB 370 / 56, 156 / 27, 60 x 512 KiB 108 / 52,
//       49 / 26, 128 x 160 KiB 47 / 38, 21 / 19.  All workgroups of 64 records read one line for their outcome, and what a record has
//       no use for costs 0.4 - 0.7 ns each (1 x 4 KiB stated as 48 MiB in 6144 workgroups 7.9, in 4096 6.4, in the form before 6.3 - 6.8), so they are
//       4096 at most; 1 x 48 MiB then takes 84 (36) us, in 6144 83 (38), in 2048 86 (41).
//   types (f32 and bf16 SUM, f16 MAX, bf16 MIN): selections of 16-bit elements need 75 - 77 vector registers, six wavefronts a
//       SIMD instead of eight, and gain alike: 530 x 32 KiB 1.06 1.14 1.27 (f16 MAX; f32 1.09 1.12 1.23), 850 0.96 1.06 1.21 (1.05 1.09 1.15), 300 x 128 KiB 1.08 1.17
//       1.33 (1.06 1.16 1.28); the least are one source of bf16 in 2900 x 8 KiB and 1240 x 16 KiB, 0.97
// A duplicate costs its first trip's payload reads: folds that are issued again whole 300 x 128 KiB from seven sources 6.2 / 27, 2900 x 4 KiB 7.9 / 20, from
// one 7.3 / 10.6; a look at the bitmap before the payload would make these 12, 8.6, 8.2 and every other call 0.4 - 0.5 us longer.
// With the size unknown, all records' first parts come first (group_place), each of 4 KiB a trip, and their number is what a call needs in which some
// records are long, us, before / this (f32 SUM of three sources; f16 MAX of one, which takes the most registers):
//   six parts, to 800 records: 260 x 4, 64 KiB 8.9 / 7.4, 25.5 / 19.5; 9.6 / 7.3, 19.2 / 16.7; 450 x 64, 128 KiB 30.4 / 29.5, 52.3 / 55.2; 22.7 / 22.6, 35.9 / 37.0;
//     450 records of 4 - 256 KiB, spread over the logarithm, 44.7 / 37.4; 37.1 / 33.9 (four parts 40.3; 39.1); 700 x 4, 64 KiB 13.3 / 8.1, 43.8 / 41.6
//   four: 900 x 4, 64, 128 KiB 15.2 / 8.7, 55.1 / 52.1, 120 / 122 (one part 8.1, 52.6, 122); 900 of 4 - 256 KiB 68.0 / 62.2; 54.3 / 53.1 (one part 102; 107);
//     1500 x 4, 128 KiB 20.4 / 11.8, 194 / 200; 2900 x 4, 16 KiB 33.7 / 21.6, 48.9 / 46.2
constexpr uint32_t kGroupFoldMost = 4096u;   // workgroups of a call of at most 160 records
static_assert(kGroupFoldMost <= 0xFFFFu, "ClaimArgs::parts");
uint32_t group_gather_parts(uint32_t n_descs, const Tuning& tune) {
  const uint32_t chunk = tune.chunk_bytes;
  if (tune.parts != 0u || n_descs > kGroupMost) return 0u;
  if (chunk == 0u) return n_descs <= 256u ? 0u : n_descs <= 800u ? 6u : 4u;
  const uint64_t bytes = static_cast<uint64_t>(n_descs) * chunk;
  if (chunk <= 8192u) {
    if (n_descs <= kGatherSmallRecords) return 0u;
    return chunk <= 4096u || n_descs > 1024u ? 1u : n_descs <= 640u ? 2u : 0u;
  }
  if (chunk <= 16384u) return chunk > 12288u && n_descs >= 550u && bytes <= (20ull << 20) ? 2u : 0u;
  if (bytes <= (16ull << 20)) return 0u;
  const bool takes = chunk <= 32768u ? bytes <= (28ull << 20) : n_descs <= 160u || (n_descs > 256u && n_descs <= 360u);
  if (!takes || bytes > (48ull << 20)) return 0u;
  const uint32_t parts = (chunk - 1u) / 8192u + 1u, most = n_descs > 160u ? parts : kGroupFoldMost / n_descs;
  return parts < most ? parts : most;
}

// Which stores a call's kernel writes through (see Through).  Lines: chunks of whole lines of 128 bytes.  Two chunks share a line where
// they are no such multiple, or their segment does not begin on one, which the host cannot see; what is shared costs more than writing through
// gives once the call has left the last-level cache.  Measured, us a pass, as the masks say / through; "odd": segments that begin off a line:
//   cut into parts, ring of 4 MiB in 64 KiB chunks 11.1 / 9.9, 32 MiB 41.4 / 39.5, odd 41.5 / 39.9, 64 MiB 67.9 / 65.2, 100 MiB (a call has 7 / 8 of it)
//     100.4 / 98.3, odd 101.5 / 99.8, 128 MiB 133.5 / 134.9, odd 134.7 / 136.5; off lines 8 MiB in 66 000-byte
//     chunks 18.2 / 16.8, 16 MiB 27.8 / 26.9, 32 MiB 43.7 / 43.8, 64 MiB 71.6 / 75.0, 128 MiB 140 / 154.  Of unknown size, chosen by record in the
//     kernel: 64 MiB in 1 MiB chunks 74.4 / 69.9, 240 MiB in 2 MiB 286 / 283, in chunks of 1 MiB and 16 bytes 79.2 / 78.3 (all written through 90.6)
//   tiles and single records (chunk_flat_kernel), the combined accumulator as before: 128 messages in 4 KiB chunks 56.5 / 55.7, 60 MiB in 4 KiB 74.0 / 73.1, odd
//     75.3 / 75.0, 80 MiB in 32 KiB 50.3 / 49.6; not the copies of a record a workgroup, which were not measured by themselves.  Copies that forward nothing, to 96 MiB:
//     all-to-all of 25 MiB in 4 KiB chunks 17.1 / 16.8, odd 17.3 / 17.0, 75 MiB 33.4 / 30.4, odd 34.8 / 31.1, 100 MiB 43.2 / 42.2, odd 44.6 / 44.5, 125 MiB 52.2 / 52.9, odd 54.3 / 58.9, 200 MiB 80.4 / 81.6,
//     odd 85.1 / 97.5, in 8 KiB 80.6 / 81.1, odd 83.3 / 96.4; those that are forwarded at any size: copy phase of 256 MiB 126.1 / 117.2, odd 131.1 / 126.6.
//     Combinations of 32-bit types to 96 MiB as well: reduce-scatter of 150 MiB 97.8 / 98.8, 256 MiB 159.9 / 161.3, odd 162.5 / 163.3, of bf16 164.5 / 161.8, in 8 KiB chunks 168.5 / 166.7
//   a workgroup a record, no staging, to 96 MiB: all-to-all in 16 KiB chunks 23.9 / 23.1, 75 MiB 30.1 / 28.0, odd 30.5 / 28.6, 88 MiB odd 35.1 / 32.4, 107 MiB 41.3 / 42.5, odd 41.8 / 46.1, 57 MiB in 32 KiB
//     odd 25.0 / 21.7; 33 008 bytes 52.9 / 55.3, 9 008 19.2 / 20.7.  With staging to 40 MiB: 38 MiB in 32 KiB odd 52.0 / 48.5, 60 MiB odd 71.0 / 76.8 (on lines 64 MiB would gain, 70.4 / 66.6)
//   decided 64 at a time: 8 x 1 MiB messages in 4 KiB chunks 27.9 / 24.9, 6 000 bytes 12 MiB 21.5 / 20.9, 30 000 bytes 22 MiB 34.3 / 35.4.  Of unknown
//     size 3.6 MB 13.3 / 12.1 and 33 MB 35.5 / 34.6, but 60 MB in 98 256-byte chunks 41.1 / 44.3: not taken.
//   in destination order, by record: 256 MiB bf16 262 / 256, 1 GiB 554 / 549, 100 MiB in 64 KiB 104 / 101, odd 256 MiB 260 / 260;
//     not copies without staging (all-to-all of 32 MiB in 64 KiB 38.9 / 39.5, where runs differ by 0.5).  With staging those of two ranks, which forward nothing, lose too (200 MiB in 64 KiB
//     70.0 / 71.2), but looking at each record for it costs the step of 256 MiB 254.8 / 256.2.  Records of unknown size are not written through: not measured
bool in_lines(const Tuning& tune) { return tune.chunk_bytes != 0u && tune.chunk_bytes % 128u == 0u; }
template <class KernelArgs>
uint64_t payload(const KernelArgs& a, const Tuning& tune) { return static_cast<uint64_t>(a.n_descs) * tune.chunk_bytes; }
constexpr uint64_t kLinesBytes = 96ull << 20;
bool few_through(const Args& a, const Tuning& tune) {   // a workgroup a record
  return in_lines(tune) && payload(a, tune) <= (a.out == nullptr ? kLinesBytes : 40ull << 20);
}
bool lines_or_small(const Args& a, const Tuning& tune) {   // decided 64 at a time, cut into parts
  return tune.chunk_bytes != 0u && payload(a, tune) <= (in_lines(tune) ? kLinesBytes : kThroughBytes);
}
bool gather_through(const GatherArgs& a, const Tuning& tune) {   // folds in tiles; see gather_store
  return tune.chunk_bytes % 128u == 0u || payload(a, tune) <= (72ull << 20);
}

// `region`: the stream's scratch words; called with its launch lock held.  HIP has no reason of its
// own to refuse a later launch of a call after it took the first: all are in one code object, their
// grids stay within 16383 * 32 workgroups of 256 threads, and a stop event that it does not take is refused with the first
// launch, which has it too.  The timing events span the whole call.
template <class KernelArgs>
int launch_ordered(void (*order)(KernelArgs, OrderArgs), void (*stream)(KernelArgs, OrderArgs), uint32_t lds, KernelArgs a, hipStream_t s,
                   const OrderPlan& o, unsigned long long* region) {
  const hipEvent_t begin = t_start, end = t_stop;
  const uint32_t n = a.n_descs;
  const auto* const descs = a.descs;
  a.parts = o.parts;
  int rc = UCCL_OK;
  for (uint32_t i = 0; i < o.launches && rc == UCCL_OK; ++i) {
    const uint32_t from = static_cast<uint32_t>(static_cast<uint64_t>(n) * i / o.launches);
    a.descs = descs + from;
    a.n_descs = static_cast<uint32_t>(static_cast<uint64_t>(n) * (i + 1u) / o.launches) - from;
    OrderArgs t;
    t.words = region;
    t.tag = g_next_tag.fetch_add(1, std::memory_order_relaxed);
    t_start = i == 0u ? begin : nullptr;
    t_stop = i == 0u ? end : nullptr;
    rc = launch_kernel(order, tiles_for(a.n_descs, kOrderThreads), kOrderThreads, s, a, t);
    if (rc != UCCL_OK) break;
    t_stop = i + 1u == o.launches ? end : nullptr;
    rc = launch_kernel_lds(stream, a.n_descs * a.parts, kOrderThreads, lds, s, a, t);
  }
  t_start = t_stop = nullptr;
  return rc;
}

template <class Op>
int launch_flat_tile(Args& a, hipStream_t s, const Tuning& tune) {
  const OrderPlan ordered = a.n_ptr == nullptr && tune.static_claims == nullptr && !tune.one_launch ? plan_ordered(a.n_descs, tune, Op::kReadsAcc, false) : kNotOrdered;
  if (ordered.launches != 0u && in_device_memory(a.descs)) {
    const Region region = claim_region(s, kOtherCalls);
    if (region.words != nullptr) {
      std::lock_guard<std::mutex> in_order(*region.launch_lock);
      // held back only where the records are known to be large: empty parts want as many workgroups as there can be
      const uint32_t lds = Op::kReadsAcc && tune.chunk_bytes != 0u ? kOrderReduceLds : 0u;
      return launch_ordered<Args>(chunk_order_kernel<Op::kEs>, in_lines(tune) && (Op::kReadsAcc || a.out != nullptr) ? chunk_ordered_kernel<Op, kAllThrough> : chunk_ordered_kernel<Op, kNoThrough>, lds, a, s, ordered, region.words);
    }
  }
  const GroupPlan grouped = a.n_ptr == nullptr && !tune.one_launch ? plan_group(a.n_descs, tune) : kNotGrouped;   // a feed's slots are pinned
  if (grouped.unroll != 0u && in_device_memory(a.descs)) {
    const Region region = claim_region(s, kGroupCalls);
    if (region.words != nullptr) {
      std::lock_guard<std::mutex> in_order(*region.launch_lock);
      a.use(region.words, region.faults);
      a.parts = grouped.parts;
      a.tag = g_next_tag.fetch_add(1, std::memory_order_relaxed);
      const bool through = lines_or_small(a, tune);
      const auto kernel = tune.chunk_bytes == 0u ? chunk_group_kernel<kGroupThreads, 4, Op, true, kNoThrough>
                          : grouped.unroll == 4u ? (through ? chunk_group_kernel<kGroupThreads, 4, Op, false, kAllThrough> : chunk_group_kernel<kGroupThreads, 4, Op, false, kNoThrough>)
                          : grouped.unroll == 2u ? (through ? chunk_group_kernel<kGroupThreads, 2, Op, false, kAllThrough> : chunk_group_kernel<kGroupThreads, 2, Op, false, kNoThrough>)
                                                 : chunk_group_kernel<kGroupThreads, 1, Op, false, kAllThrough>;   // 12 MB at most
      return launch_kernel(kernel, a.n_descs * a.parts, kGroupThreads, s, a);
    }
  }
  Plan p = plan_apply(a.n_descs, tune, Op::kReadsAcc);
  if (p.route == kRouteParts) {
    a.parts = p.parts;
    const auto launch_parts = [&](unsigned long long tag) {
      a.tag = tag;
      return launch_kernel(tune.static_claims != nullptr ? chunk_few_kernel<UCCL_PART_THREADS, UCCL_PART_UNROLL, Op, kByRecord, true, true>
                           : tune.chunk_bytes == 0u      ? chunk_few_kernel<UCCL_PART_THREADS, UCCL_PART_UNROLL, Op, kByRecord, true, false>
                           : lines_or_small(a, tune)     ? chunk_few_kernel<UCCL_PART_THREADS, UCCL_PART_UNROLL, Op, kAllThrough, true, false>
                                                         : chunk_few_kernel<UCCL_PART_THREADS, UCCL_PART_UNROLL, Op, kNoThrough, true, false>,
                           a.n_descs * p.parts, UCCL_PART_THREADS, s, a);
    };
    if (tune.static_claims != nullptr) {
      // Every call shares the device's one array and finds what other calls left there stale by their tags.
      a.use(tune.static_claims, tune.static_claims + UCCL_NOALLOC_MAX_DESCS * UCCL_CLAIM_STRIDE);
      hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
      if (hipStreamIsCapturing(s, &cap) != hipSuccess) {
        (void)hipGetLastError();
        cap = hipStreamCaptureStatusActive;   // not known: the form that is right either way
      }
      if (cap == hipStreamCaptureStatusNone) return launch_parts(g_next_tag.fetch_add(1, std::memory_order_relaxed));
      // A captured call carries the same tag in every replay, so it clears its words first, with a fill
      // kernel (no memset node); no eager call draws that tag.  (An eager call without the fill and its gap: 28 + 28
      // records of 32 KiB, reset included, 15.9 us with it, 11.2 without.)
      const hipEvent_t keep0 = t_start, keep1 = t_stop;  // the timing events belong to the data kernel
      t_start = t_stop = nullptr;
      const uint64_t words = 2ull * a.n_descs * UCCL_CLAIM_STRIDE;
      const int rc = launch_kernel(fill_words_kernel, static_cast<uint32_t>((words + 255) / 256), 256, s,
                                   reinterpret_cast<uint32_t*>(a.claims), words, 0u);
      if (rc != UCCL_OK) return rc;
      t_start = keep0;
      t_stop = keep1;
      return launch_parts(1ull);
    }
    const Region region = claim_region(s, kCutCalls);
    if (region.words != nullptr) {
      std::lock_guard<std::mutex> in_order(*region.launch_lock);
      a.use(region.words, region.faults);
      return launch_parts(g_next_tag.fetch_add(1, std::memory_order_relaxed));
    }
    a.parts = 1u;
    p.route = a.n_descs < kFewRecords ? kRouteFew : kRouteOne;   // no claim words to be had: uncut
  }
  switch (p.route) {
    case kRouteHalf:
      return launch_kernel(few_through(a, tune) ? chunk_few_kernel<1024, 1, Op, kAllThrough, false> : chunk_few_kernel<1024, 1, Op, kNoThrough, false>, a.n_descs, 1024, s, a);
    case kRouteSmall1: return launch_kernel(chunk_few_kernel<256, 1, Op, kNoThrough, false>, a.n_descs, 256, s, a);   // next to nothing to write back
    case kRouteSmall2: return launch_kernel(chunk_few_kernel<256, 2, Op, kNoThrough, false>, a.n_descs, 256, s, a);
    case kRouteFew:
      return launch_kernel(few_through(a, tune) ? chunk_few_kernel<UCCL_FEW_THREADS, UCCL_FEW_UNROLL, Op, kAllThrough, false>
                                                : chunk_few_kernel<UCCL_FEW_THREADS, UCCL_FEW_UNROLL, Op, kNoThrough, false>,
                           a.n_descs, UCCL_FEW_THREADS, s, a);
    case kRouteTile:
      if (p.tile >= 32) return launch_flat<32, UCCL_FLAT_UNROLL, Op>(a, s);
      if (p.tile >= 16) return launch_flat<16, UCCL_FLAT_UNROLL, Op>(a, s);
      if (!in_lines(tune)) return launch_tiles<Op, kNoThrough>(a, s, p.tile);
      if (payload(a, tune) > kLinesBytes) return launch_tiles<Op, !Op::kReadsAcc ? kForwarded : Op::kEs == 4 ? kNoThrough : kAllButCombined>(a, s, p.tile);
      return launch_tiles<Op, kAllButCombined>(a, s, p.tile);
    default: {
      if constexpr (Op::kReadsAcc) {
        if (in_lines(tune)) return launch_flat<1, UCCL_FLAT1_REDUCE_UNROLL, Op, kAllButCombined>(a, s);
        return launch_flat<1, UCCL_FLAT1_REDUCE_UNROLL, Op>(a, s);
      } else {
        return launch_flat<1, UCCL_FLAT_UNROLL, Op>(a, s);
      }
    }
  }
}

template <int T, class Op, Store ACC>
int launch_gather(const GatherArgs& a, hipStream_t s) {
  return launch_kernel(chunk_gather_kernel<1024, T, UCCL_GATHER_UNROLL, Op, ACC>, tiles_for(a.n_descs, T), 1024, s, a);
}
template <class Op, Store ACC>
int launch_gather_tiles(const GatherArgs& a, hipStream_t s, uint32_t tile) {
  if (tile >= 16) return launch_gather<16, Op, ACC>(a, s);
  if (tile >= 8) return launch_gather<8, Op, ACC>(a, s);
  if (tile >= 4) return launch_gather<4, Op, ACC>(a, s);
  return launch_gather<2, Op, ACC>(a, s);
}

// Workgroups per multi-source record for a call of few of them.  A record moves n + 2 streams of its
// length through one compute unit, so cutting pays from 32 KiB chunks on (measured with seven
// sources, kernel time uncut -> cut: 8 x 128 KiB 24.9 -> 6.0 us in 16 parts; 32 x 64 KiB 16.1 ->
// 6.7 us in 8; 128 x 32 KiB 12.3 -> 10.1 us in 4; 128 x 128 KiB 35.4 -> 28.1 us in 16; 512 x 32 KiB
// 32.2 -> 32.0 us in 4): parts of about 8 KiB, at most 16, while the call has at most 16 MiB of
// destination payload and the launch stays within 2048 workgroups; with the chunk size unknown, by
// record count alone.  Smaller chunks are cut into parts of 4 KiB, one vector per lane, in calls of up to 288
// records, which as tiles leave most compute units idle (event pairs, bf16, tiles -> parts; seven sources:
// 8 x 4 KiB 9.2 -> 5.5 us, 65 x 16 KiB 11.4 -> 6.4, 256 x 9 KB 14.6 -> 8.8; one source: 65 x 4 KiB 6.0 -> 4.8,
// 256 x 4 KiB 6.7 -> 6.6, but 400 x 4 KiB 7.1 -> 7.9, hence the limit).
uint32_t gather_parts(uint32_t n_descs, uint32_t chunk_bytes) {
  if (chunk_bytes == 0u) return n_descs <= 64u ? 8u : n_descs <= 128u ? 4u : 1u;
  if (static_cast<uint64_t>(n_descs) * chunk_bytes > (16ull << 20)) return 1u;
  uint32_t parts = 16u;
  while (parts > 1u && parts * kPartBytes > chunk_bytes) parts /= 2u;
  while (parts > 1u && n_descs * parts > 2048u) parts /= 2u;
  return parts;
}

Plan plan_gather_uncut(uint32_t n_descs, const Tuning& tune) {
  const uint32_t t = flat_tile(n_descs, tune.chunk_bytes);
  if (t >= 2) return {kRouteTile, t >= 16 ? 16u : t >= 8 ? 8u : t >= 4 ? 4u : 2u, 1u, 1024u, UCCL_GATHER_UNROLL};
  return {kRouteOne, 1u, 1u, 1024u, UCCL_GATHER_UNROLL};
}

Plan plan_gather(uint32_t n_descs, const Tuning& tune) {
  if (flat_tile(n_descs, tune.chunk_bytes) >= 2) {
    if (tune.chunk_bytes != 0u && tune.parts == 0u && n_descs <= kGatherSmallRecords)
      return {kRouteParts, 1u, (tune.chunk_bytes - 1u) / (UCCL_PART_THREADS * 16u) + 1u, UCCL_PART_THREADS, 1u};
  } else {
    const uint32_t parts = tune.parts ? tune.parts : gather_parts(n_descs, tune.chunk_bytes);
    if (parts > 1u && n_descs <= kRegionRecords) return {kRouteParts, 1u, parts, UCCL_PART_THREADS, UCCL_GATHER_UNROLL};
  }
  return plan_gather_uncut(n_descs, tune);
}

template <class Op>
int launch_gather_tile(GatherArgs& a, hipStream_t s, const Tuning& tune) {
  const OrderPlan ordered = plan_ordered(a.n_descs, tune, true, true);
  if (ordered.launches != 0u && in_device_memory(a.descs)) {
    const Region region = claim_region(s, kOtherCalls);
    if (region.words != nullptr) {
      std::lock_guard<std::mutex> in_order(*region.launch_lock);
      return launch_ordered<GatherArgs>(gather_order_kernel<Op::kEs>, gather_ordered_kernel<Op>, 0u, a, s, ordered, region.words);
    }
  }
  const uint32_t grouped = group_gather_parts(a.n_descs, tune);
  if (grouped != 0u && in_device_memory(a.descs)) {
    const Region region = claim_region(s, kGroupCalls);
    if (region.words != nullptr) {
      std::lock_guard<std::mutex> in_order(*region.launch_lock);
      a.use(region.words, region.faults);
      a.parts = grouped;
      a.tag = g_next_tag.fetch_add(1, std::memory_order_relaxed);
      return launch_kernel(tune.chunk_bytes == 0u ? gather_group_kernel<Op, true> : gather_group_kernel<Op, false>, a.n_descs * a.parts, 256, s, a);
    }
  }
  Plan p = plan_gather(a.n_descs, tune);
  if (p.route == kRouteParts) {
    if (p.parts == 1u) return launch_kernel(chunk_gather_parts_kernel<UCCL_PART_THREADS, 1, Op>, a.n_descs, UCCL_PART_THREADS, s, a);
    const Region region = claim_region(s, p.unroll == 1u ? kOtherCalls : kCutCalls);   // small chunks have another form that is nearly as good
    if (region.words != nullptr) {
      std::lock_guard<std::mutex> in_order(*region.launch_lock);
      a.use(region.words, region.faults);
      a.tag = g_next_tag.fetch_add(1, std::memory_order_relaxed);
      a.parts = p.parts;
      return p.unroll == 1u ? launch_kernel(chunk_gather_parts_kernel<UCCL_PART_THREADS, 1, Op>, a.n_descs * p.parts, UCCL_PART_THREADS, s, a)
                            : launch_kernel(chunk_gather_parts_kernel<UCCL_PART_THREADS, UCCL_GATHER_UNROLL, Op>, a.n_descs * p.parts,
                                            UCCL_PART_THREADS, s, a);
    }
    p = plan_gather_uncut(a.n_descs, tune);   // no claim words to be had
  }
  if (p.route != kRouteTile) return launch_gather<1, Op, kThrough>(a, s);
  return gather_through(a, tune) ? launch_gather_tiles<Op, kThrough>(a, s, p.tile) : launch_gather_tiles<Op, kCached>(a, s, p.tile);
}

bool misaligned(const void* p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) != 0; }

bool overlaps(const void* p, uint64_t pn, const void* q, uint64_t qn) {
  if (!p || !q || pn == 0 || qn == 0) return false;
  const uintptr_t a = reinterpret_cast<uintptr_t>(p), b = reinterpret_cast<uintptr_t>(q);
  return a < b + qn && b < a + pn;
}

bool tuning_from(const uccl_launch_opts* opts, Tuning* t) {
  *t = Tuning{0u, 0u, nullptr};
  if (opts == nullptr) return true;
  if (opts->parts > 16u || opts->reserved[0] != 0u || opts->reserved[1] != 0u) return false;
  *t = Tuning{opts->chunk_bytes, opts->parts, nullptr};
  return true;
}

int apply_common(void* acc, void* out_stage, const void* recv_stage, const uccl_chunk_desc* descs,
                 uint32_t n_descs, uint32_t* bitmap, int dtype, int op, bool allow_forward,
                 const uccl_extents* ext, uint32_t* n_rejected, const Tuning& tune, void* stream,
                 const uint32_t* n_ptr = nullptr) {
  if (dtype < UCCL_F32 || dtype > UCCL_I32) return UCCL_EINVAL;
  if (op < UCCL_SUM || op > UCCL_PROD) return UCCL_EINVAL;
  if (n_descs == 0) return UCCL_OK;
  if (!acc || !recv_stage || !descs || !bitmap) return UCCL_EINVAL;
  if (misaligned(acc, 16) || misaligned(out_stage, 16) || misaligned(recv_stage, 16) ||
      misaligned(descs, 16) || misaligned(bitmap, 4) || misaligned(n_rejected, 4) ||
      misaligned(n_ptr, 4))
    return UCCL_EALIGN;
  Args a;
  a.acc = static_cast<char*>(acc);
  a.out = static_cast<char*>(out_stage);
  a.recv = static_cast<const char*>(recv_stage);
  a.descs = descs;
  a.bitmap = bitmap;
  a.rejected = n_rejected;
  a.n_ptr = n_ptr;
  a.n_descs = n_descs;
  a.allow_forward = allow_forward ? 1u : 0u;
  a.claims = nullptr;
  a.faults_at = 0u;
  a.parts = 1u;
  a.tag = 0ull;
  if (ext) {
    if (overlaps(recv_stage, ext->recv_bytes, acc, ext->acc_bytes) ||
        overlaps(recv_stage, ext->recv_bytes, out_stage, ext->out_bytes) ||
        overlaps(acc, ext->acc_bytes, out_stage, ext->out_bytes))
      return UCCL_EINVAL;
    a.ext = Extents{ext->acc_bytes, out_stage ? ext->out_bytes : 0, ext->recv_bytes, ext->n_bits};
  } else {
    a.ext = Extents{UINT64_MAX, UINT64_MAX, UINT64_MAX, UINT64_MAX};
  }
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (op == UCCL_COPY) return launch_flat_tile<Copy>(a, s, tune);
  switch (dtype * 8 + op) {
    case UCCL_F32 * 8 + UCCL_SUM: return launch_flat_tile<OpF32<kSum>>(a, s, tune);
    case UCCL_F32 * 8 + UCCL_MAX: return launch_flat_tile<OpF32<kMax>>(a, s, tune);
    case UCCL_F32 * 8 + UCCL_MIN: return launch_flat_tile<OpF32<kMin>>(a, s, tune);
    case UCCL_F32 * 8 + UCCL_PROD: return launch_flat_tile<OpF32<kProd>>(a, s, tune);
    case UCCL_BF16 * 8 + UCCL_SUM: return launch_flat_tile<Op16<kSum, WidenBF16>>(a, s, tune);
    case UCCL_BF16 * 8 + UCCL_MAX: return launch_flat_tile<Op16<kMax, WidenBF16>>(a, s, tune);
    case UCCL_BF16 * 8 + UCCL_MIN: return launch_flat_tile<Op16<kMin, WidenBF16>>(a, s, tune);
    case UCCL_BF16 * 8 + UCCL_PROD: return launch_flat_tile<Op16<kProd, WidenBF16>>(a, s, tune);
    case UCCL_F16 * 8 + UCCL_SUM: return launch_flat_tile<Op16<kSum, WidenF16>>(a, s, tune);
    case UCCL_F16 * 8 + UCCL_MAX: return launch_flat_tile<Op16<kMax, WidenF16>>(a, s, tune);
    case UCCL_F16 * 8 + UCCL_MIN: return launch_flat_tile<Op16<kMin, WidenF16>>(a, s, tune);
    case UCCL_F16 * 8 + UCCL_PROD: return launch_flat_tile<Op16<kProd, WidenF16>>(a, s, tune);
    case UCCL_I32 * 8 + UCCL_SUM: return launch_flat_tile<OpI32<kSum>>(a, s, tune);
    case UCCL_I32 * 8 + UCCL_MAX: return launch_flat_tile<OpI32<kMax>>(a, s, tune);
    case UCCL_I32 * 8 + UCCL_MIN: return launch_flat_tile<OpI32<kMin>>(a, s, tune);
    case UCCL_I32 * 8 + UCCL_PROD: return launch_flat_tile<OpI32<kProd>>(a, s, tune);
    default: return UCCL_EINVAL;
  }
}

// ---- host-side batcher -------------------------------------------------------------------
//
// Appendix C.4: launching a kernel per batch is what hurts small messages, and batching
// adaptively is the remedy.  The feed collects records on the host in pinned slots and
// hands a slot to the GPU (one asynchronous copy of the records, one kernel per lane) when
// the slot is full, when the caller says so, or -- uccl_feed_poll -- as soon as the previous
// hand-over has finished, so that batches grow exactly as large as the GPU's backlog
// requires and a lone message is launched at once.  Lanes keep records of dependent phases
// apart: a flush issues lane 0 before lane 1, so a message whose reduce-scatter records go
// to lane 0 before its allgather records go to lane 1 is always applied in that order.
// Hand-overs of at most this many records per lane are read from pinned host memory directly.
#ifndef UCCL_FEED_DIRECT_RECORDS
#define UCCL_FEED_DIRECT_RECORDS 16384
#endif

struct FeedSlot {
  uccl_chunk_desc* host[2];
  uccl_chunk_desc* dev[2];
  uint32_t count[2];
  uint32_t max_len[2];  // largest payload length among the lane's records: the hand-over's chunk size
  hipEvent_t done;
  bool in_flight;
};

}  // namespace

struct uccl_feed {
  void* acc;
  void* out_stage;
  const void* recv_stage;
  uint32_t* bitmap;
  int dtype;
  int op[2];
  uint32_t capacity, n_slots, cur;
  hipStream_t stream;
  FeedSlot* slots;
  uccl_feed_stats stats;
};

namespace {

void feed_free(uccl_feed* f) {
  if (!f) return;
  if (f->slots) {
    for (uint32_t i = 0; i < f->n_slots; ++i) {
      for (int l = 0; l < 2; ++l) {
        if (f->slots[i].host[l]) (void)hipHostFree(f->slots[i].host[l]);
        if (f->slots[i].dev[l]) (void)hipFree(f->slots[i].dev[l]);
      }
      if (f->slots[i].done) (void)hipEventDestroy(f->slots[i].done);
    }
    delete[] f->slots;
  }
  delete f;
}

int feed_flush(uccl_feed* f) {
  FeedSlot& sl = f->slots[f->cur];
  const uint32_t n = sl.count[0] + sl.count[1];
  if (n == 0) return UCCL_OK;
  for (int l = 0; l < 2; ++l) {
    if (sl.count[l] == 0) continue;
    // A small batch is read by the kernel straight from the pinned slot (one bus round trip per
    // workgroup, no copy to enqueue); a large one is copied to device memory first, so that
    // thousands of workgroups do not each wait on the host bus.
    const uccl_chunk_desc* records = sl.host[l];
    const Tuning tune{sl.max_len[l], 0u, nullptr, true};
    if (sl.count[l] > UCCL_FEED_DIRECT_RECORDS) {
      const hipError_t e = hipMemcpyAsync(sl.dev[l], sl.host[l], sizeof(uccl_chunk_desc) * sl.count[l],
                                          hipMemcpyHostToDevice, f->stream);
      if (e != hipSuccess) return launch_failed(e);
      records = sl.dev[l];
    }
    const int rc = apply_common(f->acc, f->out_stage, f->recv_stage, records, sl.count[l], f->bitmap,
                                f->dtype, f->op[l], true, nullptr, nullptr, tune, f->stream);
    if (rc != UCCL_OK) return rc;
  }
  const hipError_t e = hipEventRecord(sl.done, f->stream);
  if (e != hipSuccess) return launch_failed(e);
  sl.in_flight = true;
  f->stats.flushes += 1;
  f->stats.records += n;
  if (n > f->stats.max_batch) f->stats.max_batch = n;
  sl.count[0] = sl.count[1] = 0;
  sl.max_len[0] = sl.max_len[1] = 0;
  // move on to the next slot; it may still be read by the copy of an earlier flush
  f->cur = (f->cur + 1) % f->n_slots;
  FeedSlot& nx = f->slots[f->cur];
  if (nx.in_flight) {
    if (hipEventQuery(nx.done) != hipSuccess) {
      (void)hipGetLastError();  // hipErrorNotReady is not an error here
      const hipError_t w = hipEventSynchronize(nx.done);
      if (w != hipSuccess) return launch_failed(w);
      f->stats.slot_waits += 1;
    }
    nx.in_flight = false;
  }
  return UCCL_OK;
}

}  // namespace

extern "C" {

int uccl_feed_create(uccl_feed** feed, void* acc, void* out_stage, const void* recv_stage,
                     uint32_t* dedup_bitmap, uccl_dtype dtype, uccl_op lane0_op, uccl_op lane1_op,
                     uint32_t capacity_records, uint32_t n_slots, void* stream) {
  if (!feed) return UCCL_EINVAL;
  *feed = nullptr;
  if (!acc || !recv_stage || !dedup_bitmap || capacity_records == 0 || n_slots < 2 || n_slots > 1024)
    return UCCL_EINVAL;
  if (dtype < UCCL_F32 || dtype > UCCL_I32) return UCCL_EINVAL;
  if (lane0_op < UCCL_SUM || lane0_op > UCCL_PROD || lane1_op < UCCL_SUM || lane1_op > UCCL_PROD)
    return UCCL_EINVAL;
  if (misaligned(acc, 16) || misaligned(out_stage, 16) || misaligned(recv_stage, 16) ||
      misaligned(dedup_bitmap, 4))
    return UCCL_EALIGN;
  uccl_feed* f = new (std::nothrow) uccl_feed();
  if (!f) return UCCL_ENOMEM;
  f->acc = acc;
  f->out_stage = out_stage;
  f->recv_stage = recv_stage;
  f->bitmap = dedup_bitmap;
  f->dtype = dtype;
  f->op[0] = lane0_op;
  f->op[1] = lane1_op;
  f->capacity = capacity_records;
  f->n_slots = n_slots;
  f->cur = 0;
  f->stream = static_cast<hipStream_t>(stream);
  f->stats = uccl_feed_stats{0, 0, 0, 0};
  f->slots = new (std::nothrow) FeedSlot[n_slots]();
  if (!f->slots) { feed_free(f); return UCCL_ENOMEM; }
  const size_t bytes = sizeof(uccl_chunk_desc) * static_cast<size_t>(capacity_records);
  for (uint32_t i = 0; i < n_slots; ++i) {
    for (int l = 0; l < 2; ++l) {
      if (hipHostMalloc(reinterpret_cast<void**>(&f->slots[i].host[l]), bytes, hipHostMallocDefault) != hipSuccess ||
          hipMalloc(reinterpret_cast<void**>(&f->slots[i].dev[l]), bytes) != hipSuccess) {
        (void)hipGetLastError();
        feed_free(f);
        return UCCL_ENOMEM;
      }
    }
    if (hipEventCreateWithFlags(&f->slots[i].done, hipEventDisableTiming) != hipSuccess) {
      (void)hipGetLastError();
      feed_free(f);
      return UCCL_ENOMEM;
    }
  }
  *feed = f;
  return UCCL_OK;
}

int uccl_feed_push(uccl_feed* f, int lane, const uccl_chunk_desc* host_records, uint32_t n) {
  if (!f || (lane != 0 && lane != 1) || (n > 0 && !host_records)) return UCCL_EINVAL;
  while (n > 0) {
    FeedSlot& sl = f->slots[f->cur];
    const uint32_t room = f->capacity - sl.count[lane];
    const uint32_t take = n < room ? n : room;
    memcpy(sl.host[lane] + sl.count[lane], host_records, sizeof(uccl_chunk_desc) * take);
    for (uint32_t i = 0; i < take; ++i)
      if (host_records[i].len > sl.max_len[lane]) sl.max_len[lane] = host_records[i].len;
    sl.count[lane] += take;
    host_records += take;
    n -= take;
    if (sl.count[lane] == f->capacity) {
      const int rc = feed_flush(f);
      if (rc != UCCL_OK) return rc;
    }
  }
  return UCCL_OK;
}

int uccl_feed_poll(uccl_feed* f) {
  if (!f) return UCCL_EINVAL;
  const FeedSlot& sl = f->slots[f->cur];
  if (sl.count[0] + sl.count[1] == 0) return UCCL_OK;
  const FeedSlot& prev = f->slots[(f->cur + f->n_slots - 1) % f->n_slots];
  if (prev.in_flight && hipEventQuery(prev.done) == hipErrorNotReady) {
    (void)hipGetLastError();  // "not ready" is an answer, not an error to leave behind
    return UCCL_OK;           // GPU still busy: keep batching
  }
  return feed_flush(f);
}

int uccl_feed_flush(uccl_feed* f) { return f ? feed_flush(f) : UCCL_EINVAL; }

int uccl_feed_sync(uccl_feed* f) {
  if (!f) return UCCL_EINVAL;
  const int rc = feed_flush(f);
  if (rc != UCCL_OK) return rc;
  for (uint32_t i = 0; i < f->n_slots; ++i) {
    if (f->slots[i].in_flight) {
      const hipError_t e = hipEventSynchronize(f->slots[i].done);
      if (e != hipSuccess) return launch_failed(e);
      f->slots[i].in_flight = false;
    }
  }
  return UCCL_OK;
}

int uccl_feed_get_stats(const uccl_feed* f, uccl_feed_stats* stats) {
  if (!f || !stats) return UCCL_EINVAL;
  *stats = f->stats;
  return UCCL_OK;
}

int uccl_feed_destroy(uccl_feed* f) {
  if (!f) return UCCL_EINVAL;
  int rc = UCCL_OK;
  for (uint32_t i = 0; i < f->n_slots; ++i)
    if (f->slots[i].in_flight && hipEventSynchronize(f->slots[i].done) != hipSuccess) rc = UCCL_ELAUNCH;
  feed_free(f);
  return rc;
}

}  // extern "C"

extern "C" {

int uccl_chunk_apply(void* acc, void* out_stage, const void* recv_stage,
                     const uccl_chunk_desc* descs, uint32_t n_descs, uint32_t* dedup_bitmap,
                     uccl_dtype dtype, uccl_op op, void* stream) {
  return apply_common(acc, out_stage, recv_stage, descs, n_descs, dedup_bitmap, dtype, op, true,
                      nullptr, nullptr, Tuning{0u, 0u, nullptr}, stream);
}

int uccl_chunk_apply_opts(void* acc, void* out_stage, const void* recv_stage,
                          const uccl_chunk_desc* descs, uint32_t n_descs, uint32_t* dedup_bitmap,
                          uccl_dtype dtype, uccl_op op, const uccl_extents* extents,
                          uint32_t* n_rejected, const uccl_launch_opts* opts, void* stream) {
  Tuning tune;
  if (!tuning_from(opts, &tune)) return UCCL_EINVAL;
  return apply_common(acc, out_stage, recv_stage, descs, n_descs, dedup_bitmap, dtype, op, true,
                      extents, n_rejected, tune, stream);
}

int uccl_chunk_apply_checked(void* acc, void* out_stage, const void* recv_stage,
                             const uccl_chunk_desc* descs, uint32_t n_descs,
                             uint32_t* dedup_bitmap, uccl_dtype dtype, uccl_op op,
                             const uccl_extents* extents, uint32_t* n_rejected, void* stream) {
  if (!extents) return UCCL_EINVAL;
  return apply_common(acc, out_stage, recv_stage, descs, n_descs, dedup_bitmap, dtype, op, true,
                      extents, n_rejected, Tuning{0u, 0u, nullptr}, stream);
}

int uccl_chunk_apply_indirect(void* acc, void* out_stage, const void* recv_stage,
                              const uccl_chunk_desc* descs, const uint32_t* n_descs_ptr,
                              uint32_t max_descs, uint32_t* dedup_bitmap, uccl_dtype dtype,
                              uccl_op op, const uccl_extents* extents, uint32_t* n_rejected,
                              const uccl_launch_opts* opts, void* stream) {
  if (max_descs > 0 && !n_descs_ptr) return UCCL_EINVAL;
  Tuning tune;
  if (!tuning_from(opts, &tune)) return UCCL_EINVAL;
  return apply_common(acc, out_stage, recv_stage, descs, max_descs, dedup_bitmap, dtype, op, true,
                      extents, n_rejected, tune, stream, n_descs_ptr);
}

int uccl_chunk_reduce_gather(void* acc, void* out_stage, const void* recv_stage,
                             const uccl_gather_desc* descs, uint32_t n_descs, uint32_t* dedup_bitmap,
                             uccl_dtype dtype, uccl_op op, const uccl_extents* extents,
                             uint32_t* n_rejected, const uccl_launch_opts* opts, void* stream) {
  if (dtype < UCCL_F32 || dtype > UCCL_I32) return UCCL_EINVAL;
  if (op != UCCL_SUM && op != UCCL_MAX && op != UCCL_MIN && op != UCCL_PROD) return UCCL_EINVAL;
  Tuning tune;
  if (!tuning_from(opts, &tune)) return UCCL_EINVAL;
  if (n_descs == 0) return UCCL_OK;
  if (!acc || !recv_stage || !descs || !dedup_bitmap) return UCCL_EINVAL;
  if (misaligned(acc, 16) || misaligned(out_stage, 16) || misaligned(recv_stage, 16) ||
      misaligned(descs, 16) || misaligned(dedup_bitmap, 4) || misaligned(n_rejected, 4))
    return UCCL_EALIGN;
  GatherArgs a;
  a.acc = static_cast<char*>(acc);
  a.out = static_cast<char*>(out_stage);
  a.recv = static_cast<const char*>(recv_stage);
  a.descs = descs;
  a.bitmap = dedup_bitmap;
  a.rejected = n_rejected;
  a.n_descs = n_descs;
  a.claims = nullptr;
  a.faults_at = 0u;
  a.allow_forward = 1u;
  a.tag = 0ull;
  a.parts = 1u;
  if (extents) {
    if (overlaps(recv_stage, extents->recv_bytes, acc, extents->acc_bytes) ||
        overlaps(recv_stage, extents->recv_bytes, out_stage, extents->out_bytes) ||
        overlaps(acc, extents->acc_bytes, out_stage, extents->out_bytes))
      return UCCL_EINVAL;
    a.ext = Extents{extents->acc_bytes, out_stage ? extents->out_bytes : 0, extents->recv_bytes, extents->n_bits};
  } else {
    a.ext = Extents{UINT64_MAX, UINT64_MAX, UINT64_MAX, UINT64_MAX};
  }
  hipStream_t s = static_cast<hipStream_t>(stream);
  switch (dtype * 8 + op) {
    case UCCL_F32 * 8 + UCCL_SUM: return launch_gather_tile<OpF32<kSum>>(a, s, tune);
    case UCCL_F32 * 8 + UCCL_MAX: return launch_gather_tile<OpF32<kMax>>(a, s, tune);
    case UCCL_F32 * 8 + UCCL_MIN: return launch_gather_tile<OpF32<kMin>>(a, s, tune);
    case UCCL_F32 * 8 + UCCL_PROD: return launch_gather_tile<OpF32<kProd>>(a, s, tune);
    case UCCL_BF16 * 8 + UCCL_SUM: return launch_gather_tile<Op16<kSum, WidenBF16>>(a, s, tune);
    case UCCL_BF16 * 8 + UCCL_MAX: return launch_gather_tile<Op16<kMax, WidenBF16>>(a, s, tune);
    case UCCL_BF16 * 8 + UCCL_MIN: return launch_gather_tile<Op16<kMin, WidenBF16>>(a, s, tune);
    case UCCL_BF16 * 8 + UCCL_PROD: return launch_gather_tile<Op16<kProd, WidenBF16>>(a, s, tune);
    case UCCL_F16 * 8 + UCCL_SUM: return launch_gather_tile<Op16<kSum, WidenF16>>(a, s, tune);
    case UCCL_F16 * 8 + UCCL_MAX: return launch_gather_tile<Op16<kMax, WidenF16>>(a, s, tune);
    case UCCL_F16 * 8 + UCCL_MIN: return launch_gather_tile<Op16<kMin, WidenF16>>(a, s, tune);
    case UCCL_F16 * 8 + UCCL_PROD: return launch_gather_tile<Op16<kProd, WidenF16>>(a, s, tune);
    case UCCL_I32 * 8 + UCCL_SUM: return launch_gather_tile<OpI32<kSum>>(a, s, tune);
    case UCCL_I32 * 8 + UCCL_MAX: return launch_gather_tile<OpI32<kMax>>(a, s, tune);
    case UCCL_I32 * 8 + UCCL_MIN: return launch_gather_tile<OpI32<kMin>>(a, s, tune);
    case UCCL_I32 * 8 + UCCL_PROD: return launch_gather_tile<OpI32<kProd>>(a, s, tune);
    default: return UCCL_EINVAL;
  }
}

int uccl_chunk_scatter(void* dst, const void* recv_stage, const uccl_chunk_desc* descs,
                       uint32_t n_descs, uint32_t* dedup_bitmap, void* stream) {
  return apply_common(dst, nullptr, recv_stage, descs, n_descs, dedup_bitmap, UCCL_BF16, UCCL_COPY,
                      false, nullptr, nullptr, Tuning{0u, 0u, nullptr}, stream);
}

int uccl_chunk_scatter_checked(void* dst, const void* recv_stage, const uccl_chunk_desc* descs,
                               uint32_t n_descs, uint32_t* dedup_bitmap,
                               const uccl_extents* extents, uint32_t* n_rejected, void* stream) {
  if (!extents) return UCCL_EINVAL;
  return apply_common(dst, nullptr, recv_stage, descs, n_descs, dedup_bitmap, UCCL_BF16, UCCL_COPY,
                      false, extents, n_rejected, Tuning{0u, 0u, nullptr}, stream);
}

int uccl_chunk_scatter_opts(void* dst, const void* recv_stage, const uccl_chunk_desc* descs,
                            uint32_t n_descs, uint32_t* dedup_bitmap, const uccl_extents* extents,
                            uint32_t* n_rejected, const uccl_launch_opts* opts, void* stream) {
  Tuning tune;
  if (!tuning_from(opts, &tune)) return UCCL_EINVAL;
  return apply_common(dst, nullptr, recv_stage, descs, n_descs, dedup_bitmap, UCCL_BF16, UCCL_COPY,
                      false, extents, n_rejected, tune, stream);
}

int uccl_init(void) {
  int dev = 0;
  int rc = current_device(&dev);
  unsigned long long* at = nullptr;
  if (rc == UCCL_OK) rc = device_array(g_scratch, HIP_SYMBOL(scratch), dev, &at);
  if (rc == UCCL_OK) rc = device_array(g_regions, HIP_SYMBOL(regions), dev, &at);
  return rc;
}

int uccl_chunk_apply_noalloc(void* acc, void* out_stage, const void* recv_stage,
                             const uccl_chunk_desc* descs, uint32_t n_descs, uint32_t* dedup_bitmap,
                             uccl_dtype dtype, uccl_op op, void* stream) {
  if (dtype < UCCL_F32 || dtype > UCCL_I32) return UCCL_EINVAL;
  if (op < UCCL_SUM || op > UCCL_PROD) return UCCL_EINVAL;
  if (n_descs > UCCL_NOALLOC_MAX_DESCS) return UCCL_ETOOBIG;
  if (n_descs == 0) return UCCL_OK;
  Tuning tune{0u, 0u, nullptr};
  int dev = 0;
  int rc = current_device(&dev);
  if (rc == UCCL_OK) rc = device_array(g_scratch, HIP_SYMBOL(scratch), dev, &tune.static_claims);
  if (rc != UCCL_OK) return rc;
  return apply_common(acc, out_stage, recv_stage, descs, n_descs, dedup_bitmap, dtype, op, true,
                      nullptr, nullptr, tune, stream);
}

int uccl_claim_timeouts(uint64_t* count) {
  if (!count) return UCCL_EINVAL;
  *count = 0;
  int dev = 0;
  const int rc = current_device(&dev);
  if (rc != UCCL_OK) return rc;
  unsigned long long* const base = g_regions.at[dev].load(std::memory_order_acquire);
  unsigned long long* const fixed = g_scratch.at[dev].load(std::memory_order_acquire);
  const void* const counters[] = {base != nullptr ? region_faults(base) : nullptr,   // not looked up: no split call so far
                                  fixed != nullptr ? fixed + UCCL_NOALLOC_MAX_DESCS * UCCL_CLAIM_STRIDE : nullptr};
  for (const void* c : counters) {
    if (c == nullptr) continue;
    uint32_t n = 0;
    const hipError_t e = hipMemcpy(&n, c, sizeof(n), hipMemcpyDeviceToHost);
    if (e != hipSuccess) return launch_failed(e);
    *count += n;
  }
  return UCCL_OK;
}

int uccl_chunk_segment(void* out_stage, const void* tensor, uint64_t tensor_off, uint64_t bytes,
                       uint32_t chunk_bytes, uint64_t stage_off, uint64_t slot_stride,
                       uccl_send_desc* send_descs, uint32_t conn_id, uint32_t msg_id, uint32_t first_csn,
                       void* stream) {
  if (conn_id > 255u || msg_id > 127u || chunk_bytes == 0u) return UCCL_EINVAL;
  if ((chunk_bytes & 15u) || (tensor_off & 15u) || (stage_off & 15u) || (slot_stride & 15u)) return UCCL_EALIGN;
  if (slot_stride < chunk_bytes) return UCCL_EINVAL;
  if (bytes == 0) return UCCL_OK;
  if (!out_stage || !tensor) return UCCL_EINVAL;
  if (misaligned(out_stage, 16) || misaligned(tensor, 16) || misaligned(send_descs, 8)) return UCCL_EALIGN;
  const uint64_t n_chunks = (bytes + chunk_bytes - 1) / chunk_bytes;
  if (n_chunks > 0xFFFFFFFFull) return UCCL_EINVAL;
  SegmentArgs a;
  a.stage = static_cast<char*>(out_stage) + stage_off;
  a.tensor = static_cast<const char*>(tensor) + tensor_off;
  a.descs = send_descs;
  a.bytes = bytes;
  a.slot_stride = slot_stride;
  a.stage_off = stage_off;
  a.n_chunks = n_chunks;
  a.chunk_bytes = chunk_bytes;
  a.units_per_chunk = (chunk_bytes + 2047u) / 2048u;
  a.conn_id = conn_id;
  a.msg_id = msg_id;
  a.first_csn = first_csn;
  const uint64_t groups = (n_chunks * a.units_per_chunk + 15) / 16;  // 16 units per workgroup
  if (groups > 0x7FFFFFFFull) return UCCL_EINVAL;
  return launch_kernel(segment_kernel, static_cast<uint32_t>(groups), 1024, static_cast<hipStream_t>(stream), a);
}

int uccl_dedup_reset(uint32_t* dedup_bitmap, uint64_t n_bits, void* stream) {
  if (n_bits == 0) return UCCL_OK;
  if (!dedup_bitmap) return UCCL_EINVAL;
  if (misaligned(dedup_bitmap, 4)) return UCCL_EALIGN;
  const uint64_t words = (n_bits + 31) / 32;
  const uint64_t blocks = (words + 255) / 256;
  const uint32_t grid = static_cast<uint32_t>(blocks < 4096 ? blocks : 4096);
  return launch_kernel(fill_words_kernel, grid, 256, static_cast<hipStream_t>(stream), dedup_bitmap, words, 0u);
}

int uccl_dedup_report(const uint32_t* dedup_bitmap, uint64_t n_bits, void* report,
                      uint32_t max_ranges, void* stream) {
  if (!report || (n_bits > 0 && !dedup_bitmap)) return UCCL_EINVAL;
  if (n_bits >= (1ull << 40)) return UCCL_EINVAL;
  if (misaligned(dedup_bitmap, 4) || misaligned(report, 8)) return UCCL_EALIGN;
  AckHeader* hdr = static_cast<AckHeader*>(report);
  uint64_t* ranges = reinterpret_cast<uint64_t*>(hdr + 1);
  hipStream_t s = static_cast<hipStream_t>(stream);
  // One workgroup per segment; several need scratch words to add up.  A bitmap of more than kAckMaxSegments
  // (each looks at all before it), or a stream without a region or being captured, gets the kernel of one workgroup.
  const uint64_t segments = n_bits == 0 ? 1 : (n_bits - 1) / kAckSegBits + 1;
  if (segments == 1)
    return launch_kernel(ack_segments_kernel, 1, 256, s, dedup_bitmap, n_bits, hdr, ranges, max_ranges, nullptr, 0ull);
  static_assert(kAckMaxSegments * 4 <= kRegionWords, "four words a segment");
  if (segments <= kAckMaxSegments) {
    const Region region = claim_region(s, kOtherCalls);
    if (region.words != nullptr) {
      std::lock_guard<std::mutex> in_order(*region.launch_lock);
      const unsigned long long tag = g_next_tag.fetch_add(1, std::memory_order_relaxed);
      return launch_kernel(ack_segments_kernel, static_cast<uint32_t>(segments), 256, s, dedup_bitmap, n_bits, hdr, ranges, max_ranges,
                           region.words, tag);
    }
  }
  return launch_kernel(ack_report_kernel, 1, 1024, s, dedup_bitmap, n_bits, hdr, ranges, max_ranges);
}

int uccl_message_status(uint32_t* dedup_bitmap, const uint32_t* n_chunks, uint32_t n_slots,
                        uint32_t bits_per_slot, uccl_msg_status* status, int recycle, void* stream) {
  if (bits_per_slot < 32 || bits_per_slot > 2048 || (bits_per_slot & 31u)) return UCCL_EINVAL;
  if (n_slots == 0) return UCCL_OK;
  if (n_slots > (1u << 24)) return UCCL_EINVAL;
  if (!dedup_bitmap || !n_chunks || !status) return UCCL_EINVAL;
  if (misaligned(dedup_bitmap, 4) || misaligned(n_chunks, 4) || misaligned(status, 16)) return UCCL_EALIGN;
  const uint32_t grid = (n_slots + 3) / 4;  // one wavefront per slot, four per workgroup
  return launch_kernel(message_status_kernel, grid, 256, static_cast<hipStream_t>(stream), dedup_bitmap,
                       n_chunks, n_slots, bits_per_slot / 32, reinterpret_cast<uint4*>(status),
                       recycle ? 1u : 0u);
}

int uccl_launch_plan(uint32_t n_descs, const uccl_launch_opts* opts, int gather, int reads_acc, uccl_plan* plan) {
  Tuning tune;
  if (!plan || !tuning_from(opts, &tune)) return UCCL_EINVAL;
  const Plan p = gather ? plan_gather(n_descs, tune) : plan_apply(n_descs, tune, reads_acc != 0);
  const bool few = !gather && p.route != kRouteTile && p.route != kRouteOne;
  plan->kernel = gather ? (p.route == kRouteParts ? UCCL_KERNEL_GATHER_PARTS : UCCL_KERNEL_GATHER)
                        : (few ? UCCL_KERNEL_FEW : UCCL_KERNEL_FLAT);
  plan->records_per_group = p.tile;
  plan->parts = p.parts;
  plan->threads = p.threads;
  plan->unit_bytes = 64u * 16u * p.unroll;
  const uint64_t groups = p.route == kRouteTile ? tiles_for(n_descs, p.tile) : static_cast<uint64_t>(n_descs) * p.parts;
  plan->groups = static_cast<uint32_t>(groups);
  plan->ordered = plan_ordered(n_descs, tune, gather || reads_acc, gather != 0).launches;
  plan->grouped = gather ? group_gather_parts(n_descs, tune) : plan_group(n_descs, tune).parts;
  return UCCL_OK;
}

int uccl_time_next_launch(void* start_event, void* stop_event) {
  t_start = static_cast<hipEvent_t>(start_event);
  t_stop = static_cast<hipEvent_t>(stop_event);
  return UCCL_OK;
}

const char* uccl_strerror(int code) {
  switch (code) {
    case UCCL_OK: return "ok";
    case UCCL_EINVAL: return "invalid argument";
    case UCCL_EALIGN: return "misaligned pointer";
    case UCCL_ELAUNCH: return "HIP launch failed";
    case UCCL_ENOMEM: return "out of memory";
    case UCCL_ETOOBIG: return "too many records for this entry point";
    default: return "unknown error code";
  }
}

const char* uccl_last_error_detail(void) { return t_detail; }

int uccl_version(void) { return UCCL_CHUNK_VERSION; }

}  // extern "C"
