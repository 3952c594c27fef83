// Small-M GEMM: C = A . B^T for at most 64 rows per row tile (decode-sized
// products and the expert layer's small groups), bf16 in, fp32 accumulation,
// bf16 out, the same product and rounding as the persistent kernel.
//
// With a few rows the work is bound by streaming B from HBM once (2 N K bytes
// against 2 M N K flops), so the kernel is built for memory-level parallelism
// rather than for operand reuse.  A workgroup owns a 64-column slice of C for
// its row tile; each of its four waves owns 16 of those columns and all of K.
// Both operands go from memory straight into an LDS ring (buffer_load ... lds)
// in stages of 64 k, eight lanes per whole 128-byte line of a row, with NS - 1
// stages in flight and one barrier per stage; the fragments of a stage are read
// while the one before it is computed.  What bounds it is the rate one CU
// streams at (20 to 26 GB/s from HBM) and how soon it gets there.  Before, a wave
// loaded its B fragments straight into operand registers, 64 bytes of 16 rows
// per load, half lines that the vector cache takes twice: 32 x 14336 x 4096
// (weights not in any cache) 32.2 us, now 22.0 (5.3 TB/s); 64 rows 46.7, now
// 26.2; 32 groups of 20 rows, 6144 x 7168, 495, now 418 (6.8 TB/s).  A tenth of
// it is the cache policy: B rows that one workgroup reads alone are loaded
// non-temporally (464 against 418), rows that several row tiles share are not
// (128 x 14336 x 4096 40.6 us, non-temporal 42.1).
// Each output element is one wave's MFMA chain over k in order, as in the
// persistent kernel.  Every B byte is fetched once and no tile is reused, so
// there is no placement to choose: the grid is a plain launch over the tiles.
//
// A plain problem is cut into row tiles of 16 MB rows (one tile up to 64
// rows); a grouped problem's workgroups each read a descriptor {first row,
// rows, first B row, first column}.  Where a B panel is read by several row
// tiles, the aware order runs them one after another on one XCD, so the panel
// crosses into that XCD's L2 once; the oblivious orders put them on
// neighbouring workgroups (column-major, dealt to different XCDs) or a row of
// tiles apart (row-major).
#include <hip/hip_runtime.h>

#include "internal.h"

namespace asym {
namespace {

constexpr int SK_WAVES = 4;
constexpr int SK_THREADS = 64 * SK_WAVES;
constexpr int SK_COLS = 16 * SK_WAVES;  // 64 columns per tile, 16 per wave
constexpr uint32_t kSkOOB = 0x80000000u;  // an offset past any range used here

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef unsigned v2u __attribute__((ext_vector_type(2)));

struct SkinnyParams {
  const uint16_t* A;
  const uint16_t* B;
  uint16_t* C;
  int M, N, K, lda, ldb, ldc;
  int tiles_n;        // 64-column tiles
  int row_tiles;      // plain GEMM: row tiles of 16 MB rows
  int order;          // plain GEMM: 0 aware, 1 column-major, 2 row-major
  int n_x;            // XCDs (workgroup i runs on XCD i mod n_x)
  const int4* desc;   // grouped: per workgroup {first row, rows, first B row, first column}; rows 0 = none
  int tile_cols;      // columns per column tile (a multiple of 8, at most 64)
  int ksplit;         // plain GEMM, one row tile: K ranges per column tile (1 = none)
  float* part;        // ksplit > 1: fp32 partial tiles [column tile][range][16 MB][64]
};

__device__ __forceinline__ __amdgpu_buffer_rsrc_t sk_rsrc(const void* base, uint32_t bytes) {
  const unsigned long long a = (unsigned long long)base;
  const unsigned long long u = ((unsigned long long)__builtin_amdgcn_readfirstlane((uint32_t)(a >> 32)) << 32) |
                               (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)a);
  return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(u), (short)0,
                                           (int)__builtin_amdgcn_readfirstlane(bytes), 0x00020000);
}

__device__ __forceinline__ uint32_t sk_pack(float a, float b) {
  bf16x2 v = {(__bf16)a, (__bf16)b};
  return __builtin_bit_cast(uint32_t, v);
}

constexpr int SK_KS = 64;               // k per stage: one 128-byte line of every row
constexpr int SK_ROW_BYTES = SK_KS * 2;

typedef int i32x4 __attribute__((ext_vector_type(4)));

// buffer descriptor words (uniform) for the asm loads
__device__ __forceinline__ i32x4 sk_words(const void* base, uint32_t bytes) {
  const unsigned long long a = (unsigned long long)base;
  return i32x4{(int)__builtin_amdgcn_readfirstlane((uint32_t)a), (int)__builtin_amdgcn_readfirstlane((uint32_t)(a >> 32)),
               (int)__builtin_amdgcn_readfirstlane(bytes), 0x00020000};
}

// 16 bytes per lane (byte offset voff + soff of the buffer) into LDS: lane L's
// land at lds + 16 L.  The compiler does not see these loads; they are waited
// for explicitly before the barrier that publishes a stage.  NT: non-temporal.
template <bool NT>
__device__ __forceinline__ void sk_dma(uint32_t lds, i32x4 rs, uint32_t voff, uint32_t soff) {
  if constexpr (NT)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen nt lds"
                 : : "s"(lds), "v"(voff), "s"(rs), "s"(soff) : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 : : "s"(lds), "v"(voff), "s"(rs), "s"(soff) : "memory", "m0");
}

// The last R stages of a ring, all of whose loads (LPS a wave and stage) are
// issued.  Stage J's fragments are in `cur`, stages up to END have been
// published, and `slot` is that of stage J + 1.
template <int R, int J, int LPS, int END = 0, typename Frags, typename Read, typename Mfmas, typename After>
__device__ __forceinline__ void sk_tail(Frags& cur, Frags& nxt, uint32_t slot, Read& read, Mfmas& mfmas, After& after) {
  if constexpr (J + 1 < R) {
    constexpr int NEXT = J == END ? J + (R - J) / 2 : END;
    if constexpr (NEXT != END) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((R - 1 - NEXT) * LPS) : "memory");
    read(nxt, slot);
    mfmas(cur);
    sk_tail<R, J + 1, LPS, NEXT>(nxt, cur, after(slot), read, mfmas, after);
  } else {
    mfmas(cur);
  }
}

// MB: 16-row blocks of the row tile (1, 2 or 4); NS: ring slots; ONCE: no other
// workgroup reads this one's B rows, and they are loaded non-temporally.
template <int MB, int NS, bool ONCE>
__global__ void __launch_bounds__(SK_THREADS) gemm_bf16_small_m(SkinnyParams p) {
  constexpr int A_BYTES = 16 * MB * SK_ROW_BYTES;                  // a stage of A
  constexpr uint32_t SLOT = A_BYTES + SK_COLS * SK_ROW_BYTES;      // and of B
  constexpr int LA = MB == 4 ? 2 : 1, LPS = LA + 2;                // loads per wave and stage: 8 rows each
  static_assert(NS >= 4 && (NS - 1) * LPS < 64, "the loads in flight must fit vmcnt");
  __shared__ __attribute__((aligned(1024))) unsigned char ring[NS * SLOT];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int row0, rows, brow0, ncol0, kr = 0, ctile = 0;
  if (p.desc) {
    const int4 d = p.desc[blockIdx.x];
    row0 = __builtin_amdgcn_readfirstlane(d.x);
    rows = __builtin_amdgcn_readfirstlane(d.y);
    brow0 = __builtin_amdgcn_readfirstlane(d.z);
    ncol0 = __builtin_amdgcn_readfirstlane(d.w);
    if (rows <= 0) return;
  } else {
    // plain GEMM: which (row tile r, column tile c) this workgroup computes
    const int i = blockIdx.x;
    int r, c;
    if (p.ksplit > 1) {
      // one row tile; workgroups i = c * ksplit + range
      c = i / p.ksplit;
      kr = i - c * p.ksplit;
      r = 0;
    } else if (p.order == 0) {
      // aware: the row tiles of column tile c run one after another on XCD
      // c mod n_x, so the B panel they all read crosses into that XCD's L2 once
      const int lane_x = i % p.n_x, q = i / p.n_x;
      const int cb = q / p.row_tiles;
      r = q - cb * p.row_tiles;
      c = cb * p.n_x + lane_x;
    } else if (p.order == 1) {
      c = i / p.row_tiles;  // column-major: a column's row tiles on neighbouring workgroups
      r = i - c * p.row_tiles;
    } else {
      r = i / p.tiles_n;    // row-major
      c = i - r * p.tiles_n;
    }
    if (c >= p.tiles_n || r >= p.row_tiles) return;
    row0 = r * 16 * MB;
    rows = min(16 * MB, p.M - row0);
    brow0 = 0;
    ncol0 = c * p.tile_cols;
    ctile = c;
  }
  // this wave's 16 columns (fewer, or none, at the tile's or the product's edge)
  const int n0 = ncol0 + wave * 16;
  const int tile_cols = min(p.N - ncol0, p.tile_cols);
  const int cols = max(0, min(16, tile_cols - wave * 16));

  // this workgroup's k-steps of 32: all of K, or its range of a split K
  const int steps = (p.K + 31) >> 5;
  const int per = (steps + p.ksplit - 1) / p.ksplit;
  const int ks0 = min(steps, kr * per), ks1 = min(steps, ks0 + per);
  const int k0 = ks0 * 32, k1 = min(p.K, ks1 * 32);
  const int KT = (k1 - k0 + SK_KS - 1) / SK_KS;

  // Rows past the tile read as zero (outside the resource), and so does a
  // 16-byte chunk at k >= k1 (K is a multiple of 8: a chunk is all inside or
  // all outside).  A row's chunk c lies at chunk c ^ ((row >> 1) & 7) of its
  // line, which keeps the 16 rows of a fragment read free of bank conflicts.
  // Loads: wave w takes rows 16 w .. 16 w + 15 of B (its own columns) and its
  // share of A's 2 MB blocks of 8 rows (waves 2 and 3 repeat those of 0 and 1
  // when there are two).
  const i32x4 ra = sk_words(p.A + (size_t)row0 * p.lda, (uint32_t)rows * p.lda * 2u);
  const i32x4 rb = sk_words(p.B + (size_t)(brow0 + ncol0) * p.ldb, (uint32_t)tile_cols * p.ldb * 2u);
  const int lrow = lane >> 3;
  const int ablk = MB == 1 ? wave & 1 : MB == 2 ? wave : 2 * wave;  // the wave's first block of A
  int ca[2], cb[2];
  uint32_t va[2], vb[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    ca[i] = (lane & 7) ^ ((lrow >> 1) | (((ablk + i) & 1) << 2));
    cb[i] = (lane & 7) ^ ((lrow >> 1) | (i << 2));
    va[i] = (uint32_t)(((ablk + i) * 8 + lrow) * p.lda + ca[i] * 8) * 2u;
    vb[i] = (uint32_t)((wave * 16 + i * 8 + lrow) * p.ldb + cb[i] * 8) * 2u;
  }
  const uint32_t lds0 = (uint32_t)(size_t)ring;
  const uint32_t da = __builtin_amdgcn_readfirstlane(lds0 + ablk * 1024);
  const uint32_t db = __builtin_amdgcn_readfirstlane(lds0 + A_BYTES + wave * 2048);
  auto load = [&](int t, uint32_t slot) {
    const int k = k0 + t * SK_KS;
    const uint32_t so = __builtin_amdgcn_readfirstlane(min(k, k1) * 2);  // never past the resource's end
#pragma unroll
    for (int i = 0; i < 2; ++i) sk_dma<ONCE>(db + slot + i * 1024, rb, k + cb[i] * 8 < k1 ? vb[i] : kSkOOB, so);
#pragma unroll
    for (int i = 0; i < LA; ++i) sk_dma<false>(da + slot + i * 1024, ra, k + ca[i] * 8 < k1 ? va[i] : kSkOOB, so);
  };
  const int lr = lane & 15;
  uint32_t fa[2], fb[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const uint32_t ch = (uint32_t)(((lane >> 4) | (h << 2)) ^ ((lr >> 1) & 7)) * 16u;
    fa[h] = lr * SK_ROW_BYTES + ch;
    fb[h] = A_BYTES + (wave * 16 + lr) * SK_ROW_BYTES + ch;
  }
  struct Frags {
    bf16x8 a[2][MB], b[2];
  };
  auto read = [&](Frags& f, uint32_t slot) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      f.b[h] = *reinterpret_cast<const bf16x8*>(ring + slot + fb[h]);
#pragma unroll
      for (int i = 0; i < MB; ++i)
        f.a[h][i] = *reinterpret_cast<const bf16x8*>(ring + slot + fa[h] + i * 16 * SK_ROW_BYTES);
    }
  };
  f32x4 acc[MB];
#pragma unroll
  for (int i = 0; i < MB; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto mfmas = [&](const Frags& f) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < MB; ++i)
        acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.b[h], f.a[h][i], acc[i], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  };
  // Stage t, its fragments in `cur`: publish stage t + 1 (this wave's loads of
  // it have landed; loads complete in order), read it into `nxt`, reload the
  // slot of stage t - 1 (`sl`: its reads were waited for before its MFMAs, which
  // every wave has issued by this barrier), then the MFMAs.
  auto stage = [&](int t, const Frags& cur, Frags& nxt, uint32_t sn, uint32_t sl) {
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((NS - 3) * LPS) : "memory");
    read(nxt, sn);
    load(t + NS - 1, sl);
    mfmas(cur);
  };
  // Stages past the last are not loaded: loads that only fill zeros take the
  // address unit as long as any others, and a K of a few stages paid for a ring of
  // them and for a barrier a stage.  The last R stages run without loads and with
  // four barriers, a shorter K with one.  16 x 4096 x 512 3.46 us, zero-filled
  // 4.46 (B into registers, before there was a ring, 3.55); 16 x 6144 x 4096, K in
  // 8 ranges, 14.9, 17.5 (16.2); 32 x 14336 x 4096 22.5, 24.1 (33.3).
  constexpr uint32_t RING = NS * SLOT;
  constexpr int R = NS - 1;  // stages in flight
  auto after = [](uint32_t slot) { return slot + SLOT == RING ? 0u : slot + SLOT; };
  Frags f0, f1;
  if (KT >= R) {
#pragma unroll
    for (int t = 0; t < R; ++t) load(t, t * SLOT);
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((R - 1) * LPS) : "memory");
    read(f0, 0);
    uint32_t sl = RING - SLOT, sc = 0, sn = SLOT;  // slots of stages t - 1, t, t + 1
    int t = 0;
    for (; t + R + 1 < KT; t += 2) {
      stage(t, f0, f1, sn, sl);
      const uint32_t s2 = after(sn);
      stage(t + 1, f1, f0, s2, sc);
      sl = sn;
      sc = s2;
      sn = after(s2);
    }
    if (t + R < KT) {
      stage(t, f0, f1, sn, sl);
      f0 = f1;
      sn = after(sn);
    }
    // The last R stages, all loaded, the first one's fragments in f0: a wait and
    // a barrier for half of what is in flight, then half of the rest, ...
    sk_tail<R, 0, LPS>(f0, f1, sn, read, mfmas, after);
  } else {
    for (int t = 0; t < KT; ++t) load(t, t * SLOT);
    asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
    read(f0, 0);  // (reads past the last stage are not used)
    int t = 0;
    uint32_t sn = SLOT;
    for (; t + 1 < KT; t += 2) {
      read(f1, sn);
      mfmas(f0);
      read(f0, sn + SLOT);
      mfmas(f1);
      sn += 2 * SLOT;
    }
    if (t < KT) mfmas(f0);
  }

  // in a 16x16 block the lane with row r = lane % 16 holds columns 4c..4c+3,
  // c = lane / 16; rows past the tile fall outside the resource
  const int nl = (lane >> 4) * 4;  // column inside the wave's 16
  if (p.ksplit > 1) {
    // split K: every range writes its fp32 tile; a second launch adds them
    float* mine = p.part + ((size_t)ctile * p.ksplit + kr) * (16 * MB * 64);
#pragma unroll
    for (int i = 0; i < MB; ++i)
      *reinterpret_cast<f32x4*>(mine + (i * 16 + lr) * 64 + wave * 16 + nl) = acc[i];
    return;
  }
  const __amdgpu_buffer_rsrc_t rc = sk_rsrc(p.C + (size_t)row0 * p.ldc, (uint32_t)rows * p.ldc * 2u);
  const bool vec_c = ((p.ldc & 3) == 0) && ((reinterpret_cast<uintptr_t>(p.C) & 7) == 0);
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    const f32x4 v = acc[i];
    const int m = i * 16 + lr;
    const uint32_t base = (uint32_t)(m * p.ldc + n0 + nl) * 2u;
    if (vec_c && nl + 3 < cols) {
      v2u w2;
      w2.x = sk_pack(v[0], v[1]);
      w2.y = sk_pack(v[2], v[3]);
      __builtin_amdgcn_raw_buffer_store_b64(w2, rc, base, 0, 0);
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const __bf16 h = (__bf16)v[r];
        __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(unsigned short, h), rc,
                                              nl + r < cols ? base + 2u * r : kSkOOB, 0, 0);
      }
    }
  }
}

// The sum of a split K: for each (column tile, row, 4 columns), the ranges'
// partial tiles added in range order, rounded to bf16 and stored.  One thread
// per 4 outputs.
__global__ void __launch_bounds__(256) small_m_reduce(const float* __restrict__ part, int tiles_n, int ksplit,
                                                      int tile_rows, int M, int N, uint16_t* __restrict__ C,
                                                      int ldc) {
  const long long id = (long long)blockIdx.x * 256 + threadIdx.x;
  const long long per_tile = (long long)tile_rows * 16;   // 16 groups of 4 columns per row
  if (id >= per_tile * tiles_n) return;
  const int c = (int)(id / per_tile);
  const int rem = (int)(id - (long long)c * per_tile);
  const int m = rem / 16, q = rem % 16;
  if (m >= M) return;
  const float* src = part + (size_t)c * ksplit * tile_rows * 64 + m * 64 + 4 * q;
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  for (int s = 0; s < ksplit; ++s) v += *reinterpret_cast<const f32x4*>(src + (size_t)s * tile_rows * 64);
  const int n = c * SK_COLS + 4 * q;
  uint16_t* dst = C + (size_t)m * ldc + n;
#pragma unroll
  for (int r = 0; r < 4; ++r)
    if (n + r < N) dst[r] = __builtin_bit_cast(unsigned short, (__bf16)v[r]);
}

}  // namespace

int small_m_blocks(int max_rows) {
  if (max_rows <= 16) return 1;
  if (max_rows <= 32) return 2;
  if (max_rows <= 64) return 4;
  return 0;
}

int launch_gemm_small_m(const SmallMLaunch& g, hipStream_t s) {
  SkinnyParams p;
  p.A = static_cast<const uint16_t*>(g.A);
  p.B = static_cast<const uint16_t*>(g.B);
  p.C = static_cast<uint16_t*>(g.C);
  p.M = g.M;
  p.N = g.N;
  p.K = g.K;
  p.lda = g.lda;
  p.ldb = g.ldb;
  p.ldc = g.ldc;
  if (g.tile_cols < 8 || g.tile_cols > SK_COLS || g.tile_cols % 8 || (g.ksplit > 1 && g.tile_cols != SK_COLS))
    return fail(ASYM_EINVAL, "small-M GEMM: column tiles of 8 to 64 columns (64 when split)");
  p.tile_cols = g.tile_cols;
  p.tiles_n = (g.N + g.tile_cols - 1) / g.tile_cols;
  p.row_tiles = g.row_tiles;
  p.order = g.order;
  p.n_x = g.n_x;
  p.desc = static_cast<const int4*>(g.d_desc);
  p.ksplit = g.ksplit;
  p.part = g.part;
  if (p.ksplit > 1 && (p.desc || p.row_tiles != 1 || !p.part))
    return fail(ASYM_EINVAL, "small-M GEMM: a split K needs one row tile and a workspace");
  const long long grid = g.grid;
  if (grid < 1 || grid > (1ll << 31) - 1) return fail(ASYM_EINVAL, "small-M GEMM: grid out of range");
  // One workgroup per CU of the stream's set at most: the ring takes most of a
  // CU's LDS (64 to 104 KiB of B in flight).  More workgroups than CUs: half of
  // that each, so that two share a CU and one's start overlaps the other's stream
  // (32 groups of 20 rows, 4096 x 2048: 98 us against 114 with the deep ring for
  // all).  Counted over the whole chip, a product of up to 256 workgroups ran two
  // rounds of deep rings on a masked stream, each CU idle at every start: 128 CUs,
  // 128 x 4096 x 4096 28.0 us, now 19.9; 32 x 14336 x 1024 8.6, now 7.0; 32 x
  // 14336 x 4096 31.7, now 30.5; 64 CUs, 32 x 10240 x 4096 47.9, now 45.2.
  const bool deep = grid <= g.set_cus;
#define ASYM_SMALL_M(mb, ns, once)                                                                          \
  hipLaunchKernelGGL((gemm_bf16_small_m<mb, ns, once>), dim3((unsigned)grid), dim3(SK_THREADS), 0, s, p)
#define ASYM_SMALL_M_CASE(mb, ns_deep, ns)                                       \
  case mb:                                                                       \
    if (deep && g.b_once)                                                        \
      ASYM_SMALL_M(mb, ns_deep, true);                                           \
    else if (deep)                                                               \
      ASYM_SMALL_M(mb, ns_deep, false);                                          \
    else if (g.b_once)                                                           \
      ASYM_SMALL_M(mb, ns, true);                                                \
    else                                                                         \
      ASYM_SMALL_M(mb, ns, false);                                               \
    break;
  switch (g.mb) {
    ASYM_SMALL_M_CASE(1, 14, 7)
    ASYM_SMALL_M_CASE(2, 12, 6)
    ASYM_SMALL_M_CASE(4, 9, 5)
    default:
      return fail(ASYM_EINVAL, "small-M GEMM: row blocks must be 1, 2 or 4");
  }
#undef ASYM_SMALL_M_CASE
#undef ASYM_SMALL_M
  ASYM_HIP(hipGetLastError());
  if (p.ksplit > 1) {
    const long long threads = (long long)p.tiles_n * 16 * g.mb * 16;
    hipLaunchKernelGGL(small_m_reduce, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s, g.part, p.tiles_n,
                       p.ksplit, 16 * g.mb, g.M, g.N, static_cast<uint16_t*>(g.C), g.ldc);
    ASYM_HIP(hipGetLastError());
  }
  return ASYM_OK;
}

int small_m_tile_cols() { return SK_COLS; }

}  // namespace asym
