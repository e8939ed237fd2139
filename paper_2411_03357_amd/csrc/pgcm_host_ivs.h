// Batch calls for callers inside the library that have the IVs at hand on the host.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/pgcm.h"

namespace pgcm {

// pgcm_encrypt_batch and pgcm_decrypt_verify_batch without AAD, with 96-bit IVs in pinned memory that is not
// written again before the batch has ended.  The IV of a single chunk that goes to burst_kernel is read here and
// travels in the kernel's arguments: from host memory it takes a kernel 1.5 us longer to come than the tables that
// are asked for at the same time (eight layers of 2 MiB through the pipe and its receiver, sixteen such
// calls: 163.0 -> 139.7).
int encrypt_with_host_ivs(pgcm_key_t* key, size_t n, const uint8_t* ivs, const void* const* src, const uint64_t* len,
                          void* const* dst, uint8_t* tags, hipStream_t stream);
int decrypt_with_host_ivs(pgcm_key_t* key, size_t n, const uint8_t* ivs, const void* const* src, const uint64_t* len,
                          void* const* dst, const uint8_t* tags, uint8_t* ok, hipStream_t stream);

}  // namespace pgcm
