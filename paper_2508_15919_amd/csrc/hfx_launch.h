// Host-callable launch helpers implemented next to the kernels (internal).
#pragma once
#include <hip/hip_runtime_api.h>

#include "hfx_desc.h"

namespace hfx {

hipError_t max_resident_workgroups(int head_dim, int* per_cu);
hipError_t launch_mixed_attention(const HfxHeader& header, int grid, void* desc, const void* q, const void* pool,
                                  void* ws, void* out, hipStream_t stream);
// Device address, on the current device, of the library's fixed workspace of HFX_STATIC_WS_BYTES
// (looked up once per device, then cached).
hipError_t static_workspace(void** ptr);
hipError_t launch_gather_kv(const HfxHeader& h, int n_tokens, const void* desc, const void* pool, int request,
                            void* k_out, void* v_out, hipStream_t stream);

hipError_t launch_append_kv(const HfxHeader& h, const void* desc, const void* k_new, const void* v_new, void* pool,
                            hipStream_t stream);

// Copies a host staging buffer to the device on `stream`: by a kernel from pinned memory to memory of the
// stream's GPU, by the runtime otherwise.  Either way the buffer is read when the stream gets there.
hipError_t upload(const void* host, void* device, size_t bytes, hipStream_t stream);

// Copies pages by (source, destination) id pairs: `n_pairs` of them in `host`, with room for as many in `device`.
hipError_t copy_pages(const void* host, void* device, long n_pairs, unsigned units_per_page, const void* src, void* dst, hipStream_t stream);

}  // namespace hfx
