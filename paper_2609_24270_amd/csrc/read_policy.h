// Which operands, read once by a launch, are loaded non-temporally: those of
// more bytes than the caches keep until they are read again, so that they pass
// by without pushing anything out and stream faster from HBM.  Host rules, plain
// functions of sizes.
#pragma once
#include <cstdint>

namespace asym {

// Decode attention's K and V.  Less than the memory-side cache holds (256 MiB) is
// read faster with ordinary loads when it is read again, and about as fast when
// other caches come between; from there on non-temporal loads gain more on the
// latter (a decode step's other layers do come between) than they lose on the
// former.  Measured at 32 query and 8 key/value heads, us, ordinary loads first,
// the cache just read (resident) and caches of several calls in turn (cold):
//            dense, resident  cold          pages, resident  cold
//   128 MiB   27.8   29.3     31.6  30.4     30.0   31.9     34.5  32.9
//   188 MiB   50.4   58.5     58.1  59.8     51.5   59.2     59.4  60.1
//   219 MiB   50.2   57.3     57.9  58.2                     59.9  58.8
//   256 MiB   50.0   52.6     57.6  52.9     49.4   51.9     58.1  52.7
//   288 MiB   78.4   80.4     85.8  80.9                     87.4  83.8
//   312 MiB   82.1   84.6     87.0  84.3     85.4   89.0     90.1  89.5
//   375 MiB   93.0   92.0     94.5  92.3     95.5   94.2     96.0  94.9
//   512 MiB  103.0   92.7    103.0  93.3    105.5   94.3    104.4  94.5
// Pages placed on the die that reads them gain the most from the caches: 128 MiB,
// resident, 26.5 and 32.6 on the whole chip, 48.6 and 62.5 on one die.
inline bool attn_streams_kv(int64_t kv_bytes) { return kv_bytes >= (256ll << 20); }

// The bytes of K and V behind a paged call: `read` over all its requests, but no
// more than the pools hold, once if both are one.  Requests that share a prefix
// name the same pages, which each of them finds in the caches: 64 requests, 8
// heads, 4096 tokens (1 GiB read) over the pages of one request, 97.8 us, and
// loaded non-temporally 135.8.
inline int64_t paged_kv_bytes(int64_t read, int64_t pool_bytes, bool one_pool) {
  const int64_t pools = one_pool ? pool_bytes : 2 * pool_bytes;
  return read < pools ? read : pools;
}

// Only where nearly the whole chip reads them: on fewer CUs the waves in flight,
// not HBM, bound the call, and each wave waits longer for a load that passes by
// the caches.  Measured, us, ordinary loads first, 16 requests x 8000 tokens of 8
// heads / 64 x 8000 of 8 / 16 x 4000 of 32: 64 CUs 218 243 / 806 930 / 365 454,
// 128 CUs 121 135 / 444 511 / 213 251, 192 CUs 129 135 / 382 402 / 231 251, 224
// CUs 136 132 / 408 404 / 242 253, 240 CUs 134 126 / 412 406 / 239 233.
inline bool attn_set_streams(int set_cus, int device_cus) { return 16 * set_cus >= 15 * device_cus; }

// Paged K and V past that line are loaded with ordinary loads all the same where
// `tasks` (one a wave) are a second round of 1/8 to 5/8 of the `round` waves that
// run at a time, and one or two query heads read a key/value head: a wave of that
// thin round waits longer for each load that passes by the caches, and more heads,
// or more waves, cover it.  Measured, us, ordinary loads first, 1 / 2 / 4 query
// heads, 64 key/value heads in all: 1.06 rounds 128.9 129.1 / 131.4 129.9 / 138.8
// 131.6, 1.25 144.3 145.7 / 146.8 146.8 / 151.5 148.9, 1.375 151.6 155.0 / 154.1
// 156.2 / 159.3 159.1, 1.56 157.0 158.9 / 159.4 159.7 / 164.4 162.4, 1.66 161.9
// 160.6 / 164.2 161.9 / 168.1 164.4, 1.78 172.0 163.7; 1.25 rounds of full splits,
// one query head, 147 and 151 to 153 (dense 143 and 141: the rule is for pages).
inline bool pages_thin_round(int heads_per_kv, int64_t tasks, int64_t round) {
  const int64_t last = tasks - round;
  return heads_per_kv <= 2 && 8 * last > round && 8 * last <= 5 * round;
}

// B of a small-M product whose rows one workgroup each reads: `bytes` of it, at
// b with a pitch of ldb bf16 values, in k ranges of `range_steps` 32-wide steps
// (0: K is not split).  Only where every stage of 64 k is a whole 128-byte line of
// each row: of a line that two stages share, the second half is gone from the
// caches when the next stage asks for it.  And only from 64 MiB on.  Measured, us,
// ordinary loads first, weights just read (resident) and several weights in turn
// (cold); a program's other weights pass through the memory-side cache between two
// launches, so the cold figures decide:
//                                        resident     cold
//   32 x 6144 x 4096        48 MiB       14.0  16.5   16.5  17.0
//   32 x 14336 x 4096      112 MiB       19.4  21.9   25.8  23.6
//   64 x 14336 x 4096      112 MiB       20.4  27.7   29.2  28.0
//   32 x 20480 x 4096      160 MiB       26.4  30.2   34.6  31.8
//   8 groups of 20 rows, 4096 x 2048
//                          128 MiB       21.0  25.6   29.6  27.2
//   32 groups of them      512 MiB       99.5  91.4   99.7  91.2
//   rows of 4088 values, half lines: 32 x 20000 x 4088
//                          156 MiB       26.3  45.3   44.6  47.4
//   32 groups of 20 rows, 1000 x 2040
//                          125 MiB       23.2  34.6   31.5  34.1
// A copy that the launch before has just written (`fresh`: the transpose of B
// stored [K][N]) is still in the memory-side cache while it and its source fit
// there.  Whole calls, us, ordinary loads first, several weights in turn:
//   32 x 4096 x 14336       112 MiB       61.0  70.9   (64 rows 63.1  77.0)
//   32 x 14336 x 4096       112 MiB       58.3  61.8   (64 rows 59.9  65.2)
//   16 x 8192 x 8192        128 MiB       74.7  74.3   (resident 74.5  70.4)
//   16 x 20480 x 4096       160 MiB       90.1  90.9
//   32 x 30000 x 4096       234 MiB      167.8 150.1
inline bool small_m_streams_b(const void* b, int64_t ldb, int64_t bytes, int64_t range_steps, bool fresh = false) {
  const bool lines = (reinterpret_cast<uintptr_t>(b) & 127u) == 0 && ldb % 64 == 0 && range_steps % 2 == 0;
  return lines && bytes >= ((fresh ? 128ll : 64ll) << 20);
}

}  // namespace asym
