// Small device functions that the HSTU kernels of both element types share.
#pragma once

#include "kernels.h"

namespace racer {

#if defined(__HIPCC__)
__device__ __forceinline__ float silu(float x) { return x / (1.0f + __expf(-x)); }

__device__ __forceinline__ uint32_t time_bucket(long long dt, uint32_t n_time) {
  const unsigned long long v = dt > 1 ? static_cast<unsigned long long>(dt) : 1ull;
  const uint32_t b = 63u - static_cast<uint32_t>(__clzll(static_cast<long long>(v)));
  return b < n_time - 1 ? b : n_time - 1;
}

// byte offset of the K (kv = 0) or V (kv = 1) block of (layer, head) inside a page
__device__ __forceinline__ uint64_t kv_block_offset(const HstuDims& hd, uint32_t layer, uint32_t kv, uint32_t head,
                                                    uint32_t esize) {
  return ((static_cast<uint64_t>(layer) * 2 + kv) * hd.H + head) * hd.pt * hd.dh * esize;
}

// page index and offset inside the page of token j (page_tokens is usually a power of two)
__device__ __forceinline__ void split_token(const HstuDims& hd, uint32_t j, uint32_t* page_idx, uint32_t* in_page) {
  if (hd.pt_shift < 32) {
    *page_idx = j >> hd.pt_shift;
    *in_page = j & (hd.pt - 1);
  } else {
    *page_idx = j / hd.pt;
    *in_page = j % hd.pt;
  }
}

// the request a new-token row belongs to, searched among requests lo .. hi (the last one that starts at or before it)
__device__ __forceinline__ uint32_t request_of(const ReqDev* reqs, uint32_t row, uint32_t lo, uint32_t hi) {
  while (lo < hi) {
    const uint32_t mid = (lo + hi + 1) / 2;
    if (reqs[mid].x_off <= row) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}
#endif

}  // namespace racer
