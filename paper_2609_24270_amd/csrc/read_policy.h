// Which operands, read once by a launch, are loaded non-temporally: those of
// more bytes than the caches keep until they are read again, so that they pass
// by without pushing anything out and stream faster from HBM.  Host rules, plain
// functions of sizes.
#pragma once
#include <cstdint>

namespace asym {

// Decode attention's K and V.  A cache that the memory-side cache (256 MiB) and
// the L2s hold is read faster with ordinary loads when it is read again; past 5/4
// of the former too little of it is left.  Measured at 32 query and 8 key/value
// heads, us, ordinary loads first, the cache just read (resident) and caches of
// several calls in turn (cold):
//            dense, resident  cold          pages, resident  cold
//   128 MiB   27.8   29.3     31.6  30.4     30.0   31.9     34.5  32.9
//   188 MiB   50.4   58.5     58.1  59.8     51.5   59.2     59.4  60.1
//   256 MiB   50.0   52.6     57.6  52.9     49.4   51.9     58.1  52.7
//   312 MiB   82.1   84.6     87.0  84.3     85.4   89.0     90.1  89.5
//   375 MiB   93.0   92.0     94.5  92.3     95.5   94.2     96.0  94.9
//   512 MiB  103.0   92.7    103.0  93.3    105.5   94.3    104.4  94.5
// Pages placed on the die that reads them gain the most from the caches: 128 MiB,
// resident, 26.5 and 32.6 on the whole chip, 48.6 and 62.5 on one die.
inline bool attn_streams_kv(int64_t kv_bytes) { return kv_bytes > (320ll << 20); }

// The bytes of K and V behind a paged call: `read` over all its requests, but no
// more than the pools hold, once if both are one.  Requests that share a prefix
// name the same pages, which each of them finds in the caches: 64 requests, 8
// heads, 4096 tokens (1 GiB read) over the pages of one request, 97.8 us, and
// loaded non-temporally 135.8.
inline int64_t paged_kv_bytes(int64_t read, int64_t pool_bytes, bool one_pool) {
  const int64_t pools = one_pool ? pool_bytes : 2 * pool_bytes;
  return read < pools ? read : pools;
}

}  // namespace asym
