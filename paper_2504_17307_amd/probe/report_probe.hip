// Measurement and test aid, not part of the product: the acknowledgement report's kernel of many workgroups, built so
// that no workgroup waits for another's counts (UCCL_ACK_POLLS 0).  Every one counts the segments before it
// itself, which in the library only happens when a workgroup is not found to have run for a long time.
#define UCCL_ACK_POLLS 0
#pragma clang diagnostic ignored "-Wunused-function"   // the other kernels of that file
#include "uccl_feedback_kernels.hpp"

// As uccl_dedup_report; words: DEVICE scratch, 4 * 8 bytes for each 32768 bits.  1 .. 2^28 bits.  Returns 0, or -1 for
// bad arguments / a refused launch.
extern "C" int uccl_probe_report(const uint32_t* bitmap, uint64_t n_bits, void* report, uint32_t max_ranges, uint64_t* words,
                                 void* stream) {
  if (!bitmap || !report || !words || n_bits == 0 || n_bits > static_cast<uint64_t>(kAckMaxSegments) * kAckSegBits) return -1;
  AckHeader* hdr = static_cast<AckHeader*>(report);
  ack_segments_kernel<<<dim3(static_cast<uint32_t>((n_bits - 1) / kAckSegBits + 1)), dim3(256), 0, static_cast<hipStream_t>(stream)>>>(
      bitmap, n_bits, hdr, reinterpret_cast<uint64_t*>(hdr + 1), max_ranges, reinterpret_cast<unsigned long long*>(words), 1ull);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}
