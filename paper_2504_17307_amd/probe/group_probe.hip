// Measurement and test aid, not part of the product: the kernels that decide 64 records at a time, built so that the first
// workgroup of a group waits like the others (UCCL_GROUP_LEADS 0) and whoever has polled twice decides.  In the library
// that only happens when a group's first workgroup has not run for a long time.  late_probe.hip builds them once more, with a
// first workgroup that begins when another has taken its place.
#ifndef UCCL_GROUP_LEADS
#define UCCL_GROUP_LEADS 0
#define UCCL_PROBE(name) name
#endif
#define UCCL_GROUP_POLLS 2
#pragma clang diagnostic ignored "-Wunused-function"   // the other kernels of that file
#include "uccl_data_kernels.hpp"

namespace {
template <class GroupArgs, class Desc>
bool probe_args(GroupArgs& a, void* acc, void* out, const void* recv, const void* descs, uint32_t n, uint32_t* bitmap, uint64_t n_bits, uint32_t* rejected,
                uint32_t parts, uint64_t* words, uint64_t tag) {
  if (!acc || !recv || !descs || !bitmap || !words || n == 0 || n > (1u << 20) || parts == 0 || parts > 64 || tag == 0) return false;
  a = {};
  a.acc = static_cast<char*>(acc);
  a.out = static_cast<char*>(out);
  a.recv = static_cast<const char*>(recv);
  a.descs = static_cast<const Desc*>(descs);
  a.bitmap = bitmap;
  a.rejected = rejected;
  a.ext = Extents{UINT64_MAX, UINT64_MAX, UINT64_MAX, n_bits};
  a.n_descs = n;
  a.allow_forward = 1u;
  a.use(reinterpret_cast<unsigned long long*>(words), words + static_cast<size_t>((n - 1) / kGroup + 1) * UCCL_CLAIM_STRIDE);
  a.tag = tag;
  a.parts = parts;
  return true;
}
int launched() { return hipGetLastError() == hipSuccess ? 0 : -1; }
}  // namespace

// fp32 SUM as uccl_chunk_apply with n_rejected, `parts` workgroups of 256 threads a record, `unroll` (1 or 4) x 4 KiB a trip; every
// group has a record that is valid and not empty, or it may stay undecided.  words: DEVICE scratch, 128 bytes for every 64 records
// and a line more, whose first word counts wavefronts that gave up.  Returns 0, or -1 for bad arguments / a refused launch.
extern "C" int UCCL_PROBE(uccl_probe_group_apply)(void* acc, void* out, const void* recv, const void* descs, uint32_t n, uint32_t* bitmap, uint64_t n_bits,
                                                  uint32_t* rejected, uint32_t parts, uint32_t part_major, uint32_t unroll, uint64_t* words, uint64_t tag,
                                                  void* stream) {
  Args a;
  if ((unroll != 1u && unroll != 4u) || part_major > 1u ||
      !probe_args<Args, uccl_chunk_desc>(a, acc, out, recv, descs, n, bitmap, n_bits, rejected, parts, words, tag))
    return -1;
  using Sum = OpF32<kSum>;
  const auto kernel = unroll == 1u ? (part_major ? chunk_group_kernel<256, 1, Sum, true, kNoThrough> : chunk_group_kernel<256, 1, Sum, false, kAllThrough>)
                                   : (part_major ? chunk_group_kernel<256, 4, Sum, true, kNoThrough> : chunk_group_kernel<256, 4, Sum, false, kAllThrough>);
  kernel<<<dim3(n * parts), dim3(256), 0, static_cast<hipStream_t>(stream)>>>(a);
  return launched();
}

// The same for fp32 SUM folds, 4 KiB a trip.
extern "C" int UCCL_PROBE(uccl_probe_group_fold)(void* acc, void* out, const void* recv, const void* descs, uint32_t n, uint32_t* bitmap, uint64_t n_bits,
                                                 uint32_t* rejected, uint32_t parts, uint32_t part_major, uint64_t* words, uint64_t tag, void* stream) {
  GatherArgs a;
  if (part_major > 1u || !probe_args<GatherArgs, uccl_gather_desc>(a, acc, out, recv, descs, n, bitmap, n_bits, rejected, parts, words, tag)) return -1;
  const auto kernel = part_major ? gather_group_kernel<OpF32<kSum>, true> : gather_group_kernel<OpF32<kSum>, false>;
  kernel<<<dim3(n * parts), dim3(256), 0, static_cast<hipStream_t>(stream)>>>(a);
  return launched();
}

extern "C" int UCCL_PROBE(uccl_probe_group)(void* acc, void* out, const void* recv, const void* descs, uint32_t n, uint32_t* bitmap, uint64_t n_bits,
                                            uint32_t* rejected, uint32_t parts, uint64_t* words, uint64_t tag, void* stream) {
  return UCCL_PROBE(uccl_probe_group_apply)(acc, out, recv, descs, n, bitmap, n_bits, rejected, parts, 0, 1, words, tag, stream);
}
