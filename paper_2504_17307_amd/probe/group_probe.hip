// Measurement and test aid, not part of the product: the kernel that decides 64 records at a time, built so that the first
// workgroup of a group waits like the others (UCCL_GROUP_LEADS 0) and whoever has polled twice decides.  In the library
// that only happens when a group's first workgroup has not run for a long time.
#define UCCL_GROUP_LEADS 0
#define UCCL_GROUP_POLLS 2
#pragma clang diagnostic ignored "-Wunused-function"   // the other kernels of that file
#include "uccl_data_kernels.hpp"

// fp32 SUM as uccl_chunk_apply with n_rejected, `parts` workgroups of 256 threads a record, 4 KiB a trip; every group has a
// record that is valid and not empty, or it stays undecided.  words: DEVICE scratch, 128 bytes for every 64 records and a
// line more, whose first word counts wavefronts that gave up.  Returns 0, or -1 for bad arguments / a refused launch.
extern "C" int uccl_probe_group(void* acc, void* out, const void* recv, const void* descs, uint32_t n, uint32_t* bitmap, uint64_t n_bits,
                                uint32_t* rejected, uint32_t parts, uint64_t* words, uint64_t tag, void* stream) {
  if (!acc || !recv || !descs || !bitmap || !words || n == 0 || n > (1u << 20) || parts == 0 || parts > 16 || tag == 0) return -1;
  Args a = {};
  a.acc = static_cast<char*>(acc);
  a.out = static_cast<char*>(out);
  a.recv = static_cast<const char*>(recv);
  a.descs = static_cast<const uccl_chunk_desc*>(descs);
  a.bitmap = bitmap;
  a.rejected = rejected;
  a.ext = Extents{UINT64_MAX, UINT64_MAX, UINT64_MAX, n_bits};
  a.n_descs = n;
  a.allow_forward = 1u;
  a.use(reinterpret_cast<unsigned long long*>(words), words + static_cast<size_t>((n - 1) / kGroup + 1) * UCCL_CLAIM_STRIDE);
  a.tag = tag;
  a.parts = parts;
  chunk_group_kernel<256, 1, OpF32<kSum>><<<dim3(n * parts), dim3(256), 0, static_cast<hipStream_t>(stream)>>>(a);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}
