// Multi-head latent attention, decode (the MLA workloads of Section 7.1;
// Appendix F counts one compressed row of 512 + 64 values per token).  Each
// request caches one 576-wide row per token, Kc[t] = [c_t (512) ; r_t (64)];
// every query head h has a 576-wide query (the projections absorbed into it):
//
//   O[b, h] = softmax_t(scale * <q[b, h], Kc[b, t]>) . Kc[b, t, 0:512]
//
// All query heads read the same rows, so the rows are the data a placement
// can share: the paper's topology-plus-locality experiment is MLA decode.
//
// Work is split along the sequence (flash-decoding).  A task is one
// (request, split, block of 16 query heads) and runs on one wave:
//   * scores S^T (16 tokens x 16 heads) = K . Q^T on the matrix cores
//     (v_mfma_f32_16x16x32_bf16, 18 steps over the 576 values): the key
//     fragment of a lane is 16 contiguous bytes of one row, loaded from memory
//     straight into operand registers; the 16 query rows stay in registers
//     for the whole task;
//   * an online softmax per head (a lane's accumulators all belong to one
//     head, so the rescaling is a per-lane factor);
//   * O^T (512 x 16 heads) += V^T . P^T on the matrix cores
//     (v_mfma_f32_16x16x16_bf16): a lane's probabilities (4 consecutive
//     tokens, one head) are already the B operand of that product; the
//     values are written to a per-wave LDS tile as they are, one 16-byte
//     store per key fragment already loaded (the latent part of the row is
//     the value, so the rows are read from memory once), and the A operand
//     V^T comes out of it through gfx950's transposing LDS read
//     (ds_read_b64_tr_b16), one per 16 values; token rows are padded by 32
//     bytes so that the reads of 16 rows spread over the banks;
//   * 16-token blocks; the next block's rows go out as soon as a block's
//     fragments are consumed (scores computed, values written), and the
//     output is rescaled only when a head's block maximum exceeds the
//     reference maximum by more than a fixed gap (the reference then follows;
//     below the gap the stale reference keeps the result exact);
//   * multiples of 64 heads run in the workgroup forms instead: four waves, each
//     on one or two head blocks, share each block's rows through LDS tiles.
// Each task writes its unnormalised output, max and sum (fp32); a second
// kernel merges the splits of each (request, head) in an order fixed by the
// split count (several waves per row when there are many splits), so the
// result does not depend on which wave ran which task.
//
// Placement.  Tasks are numbered in one of two orders.  Aware: request-split
// major, the head blocks of one (request, split) consecutive; each XCD gets a
// share of that list in proportion to its CUs in the stream's set, and its
// workgroups claim groups of 4 tasks from it, then from the other shares, so
// the head blocks that read the same rows run on one XCD, close in time (the
// rows cross into its L2 once).  Oblivious: head-block major (a grid over
// heads, then requests and splits), 4 tasks per workgroup in order; the
// hardware deals workgroups round-robin, so the head blocks of one split
// land on different XCDs and each XCD gets the same share whatever its CUs.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "internal.h"
#include "split_merge.h"

namespace asym {
namespace {

constexpr int MD = 576;            // query / key width
constexpr int MV = 512;            // value (latent) width
constexpr int MW = 4;              // tasks per workgroup, one per wave
constexpr int MT = 16;             // tokens per block
constexpr int MSTEPS = MD / 32;    // 18 MFMA steps for the scores
constexpr int VSTEPS = MV / 32;    // 16 of them cover the latent part
constexpr int V_ROW = MV * 2 + 32;  // bytes of one token's values in the per-wave tile, padded
constexpr int V_BYTES = MT * V_ROW;  // 16.5 KiB per wave
constexpr int MG = 4;              // workgroup forms: waves, each on one or two head blocks
constexpr int MT2 = 32;            // workgroup forms: tokens per block
constexpr int T2_GROUPS = MD / 64;   // workgroup forms: 128-byte pieces of a row
constexpr int T2_GROUP_BYTES = MT2 * 128;  // one piece of the block's 32 rows
constexpr int T2_BYTES = T2_GROUPS * T2_GROUP_BYTES;  // 36 KiB per tile, four tiles
constexpr int T2_TILES = 4;
constexpr uint32_t kMlOOB = 0x80000000u;
constexpr int kMlClaimStride = 64;  // ints between claim counters (256-byte lines)

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef short i16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) unsigned char lds_u8;
typedef __attribute__((address_space(3))) const bf16x8 lds_bf16x8;
typedef __attribute__((address_space(3))) i16x4 lds_i16x4;

struct MlaParams {
  const uint16_t* q;     // [B][Hq][576]
  const uint16_t* kv;    // [B][S][576]
  float* part_o;         // [B][Hq][n_splits][512]
  float* part_ml;        // [B][Hq][n_splits][2]: max, sum
  const int* quota_off;  // aware: [n_x + 1] start of each XCD's share (tasks); null = oblivious
  int* claim;            // aware: groups of 4 claimed from share y at claim[y * kMlClaimStride]
  uint32_t allow;        // aware: XCDs whose workgroups may work
  int B, Hq, S, split, n_splits, hblocks, tasks, n_x;
  float scale;
};

__device__ __forceinline__ __amdgpu_buffer_rsrc_t ml_rsrc(const void* base, uint32_t bytes) {
  const unsigned long long a = (unsigned long long)base;
  const unsigned long long u = ((unsigned long long)__builtin_amdgcn_readfirstlane((uint32_t)(a >> 32)) << 32) |
                               (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)a);
  return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(u), (short)0,
                                           (int)__builtin_amdgcn_readfirstlane(bytes), 0x00020000);
}

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// (request, split, head block) of task i in either order.
__device__ __forceinline__ void mla_task_of(const MlaParams& p, bool aware, int i, int& b, int& split, int& hb) {
  if (aware) {
    hb = i % p.hblocks;
    const int r = i / p.hblocks;
    split = r % p.n_splits;
    b = r / p.n_splits;
  } else {
    const int bs = p.B * p.n_splits;
    hb = i / bs;
    const int r = i - hb * bs;
    split = r % p.n_splits;
    b = r / p.n_splits;
  }
}

// The maximum over the four lanes l, l ^ 16, l ^ 32, l ^ 48: each row swap
// (v_permlane16_swap, v_permlane32_swap) of a value with itself leaves every
// lane the pair {x[l], x[l ^ 16]} (then ^ 32) in its two results; in the
// vector unit, with no LDS round trip.  A maximum is exact in any order.
__device__ __forceinline__ float ml_max4(float x) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// ---- the arithmetic of one 16-token block, shared by both forms ----------
// Scores S^T (16 tokens x 16 heads) = K . Q^T: lane (lr, lq) gets tokens
// 4 lq .. 4 lq + 3 of the block, head lr.
__device__ __forceinline__ f32x4 mla_scores(const bf16x8 (&kf)[MSTEPS], const bf16x8 (&qf)[MSTEPS]) {
  f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < MSTEPS; ++c) s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[c], qf[c], s, 0, 0, 0);
  return s;
}

// Online softmax of a block (tokens past t1 masked): updates the reference
// max and the sum, rescales the output when some head's block maximum exceeds
// its reference by more than kRescaleGap (the factor is exactly 1 elsewhere)
// and returns the probabilities, relative to the reference, as the B operand
// of P.V.  A reference below the true maximum leaves the result exact (the
// output, the sum and the max that the merge receives all use it); it only
// lets probabilities reach e^kRescaleGap, and saves the 128-multiply rescale
// on most blocks (with the exact maximum, a random sequence raised some head's
// maximum on about 60% of the blocks of a 1024-token split).
constexpr float kRescaleGap = 8.f;
__device__ __forceinline__ i16x4 mla_softmax(f32x4 s, int tok0, int t1, float scale, int lq, f32x4 (&o)[MV / 16],
                                             float& m_run, float& l_part) {
  float v[4];
  float bm = -INFINITY;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int tok = tok0 + 4 * lq + i;
    v[i] = tok < t1 ? s[i] * scale : -INFINITY;
    bm = fmaxf(bm, v[i]);
  }
  bm = ml_max4(bm);
  // bm is finite (every block has a token); the first block always raises
  const bool raise = bm > m_run + kRescaleGap;
  const float m_new = raise ? bm : m_run;
  const float alpha = raise ? __expf(m_run - m_new) : 1.f;
  m_run = m_new;
  float pr[4];
  float ps = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    pr[i] = __expf(v[i] - m_new);
    ps += pr[i];
  }
  l_part = l_part * alpha + ps;
  i16x4 pb;
#pragma unroll
  for (int i = 0; i < 4; ++i) pb[i] = __builtin_bit_cast(short, (__bf16)pr[i]);
  if (__ballot(raise)) {
#pragma unroll
    for (int j = 0; j < MV / 16; ++j) o[j] *= alpha;
  }
  return pb;
}

// O^T (512 values x 16 heads) += V^T . P^T from a row-major tile (token rows
// of `pitch` bytes, the latent values first).  The A operand
// V^T[16 j + lr][4 lq .. 4 lq + 3] comes from a transposing read: in each
// group of 16 lanes, result lane r takes element r % 4 of the 8 bytes that
// lanes 4 i + r / 4 address, i = 0 .. 3; lane (lr, lq) addresses token
// 4 lq + lr / 4, values 16 j + 4 (lr % 4) .. + 3.  In batches of 8, the next
// batch's reads in flight while a batch's MFMAs run (an empty asm that takes a
// whole batch keeps the compiler from placing each read next to its use).
__device__ __forceinline__ void mla_pv(const unsigned char* tile, uint32_t pitch, i16x4 pb, int lr, int lq,
                                       f32x4 (&o)[MV / 16]) {
  const uint32_t tr0 = (uint32_t)(4 * lq + (lr >> 2)) * pitch + 8u * (lr & 3);
  auto read_batch = [&](int jb, i16x4 (&a)[8]) {
#pragma unroll
    for (int u = 0; u < 8; ++u)
      a[u] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
          (__attribute__((address_space(3))) i16x4*)(tile + tr0 + 32u * (jb + u)));
  };
  i16x4 ab[2][8];
  read_batch(0, ab[0]);
#pragma unroll
  for (int jb = 0; jb < MV / 16; jb += 8) {
    i16x4 (&cur)[8] = ab[(jb / 8) & 1];
    asm volatile("" : "+v"(cur[0]), "+v"(cur[1]), "+v"(cur[2]), "+v"(cur[3]), "+v"(cur[4]), "+v"(cur[5]),
                 "+v"(cur[6]), "+v"(cur[7]));
    if (jb + 8 < MV / 16) read_batch(jb + 8, ab[((jb / 8) + 1) & 1]);
#pragma unroll
    for (int u = 0; u < 8; ++u) o[jb + u] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(cur[u], pb, o[jb + u], 0, 0, 0);
  }
}

// The workgroup form's block of 32 tokens, as two 16-token halves: s0 and
// s1 give lane (lr, lq) tokens 4 lq .. 4 lq + 3 and 16 + 4 lq .. 16 + 4 lq + 3
// of head lr.  The softmax step is that of mla_softmax over the 32 tokens;
// the probabilities come back as the B operand of a 32-deep product whose
// k index 8 lq + i stands for the first group's token 4 lq + i (i < 4) and
// the second group's token 16 + 4 lq + i - 4 (i >= 4).
// In steps, so that a caller can put them between other work; `alpha` is the
// factor the output takes when the wave's ballot of `raise` is set (exactly 1
// on other lanes).
struct Softmax32 {
  float v[8], ps;
  bf16x8 pb;
  float alpha;
  bool raise;
  // the scaled scores, tokens from t1 on masked (only the last block has any)
  __device__ __forceinline__ void scores(f32x4 s0, f32x4 s1, int tok0, int t1, float scale, int lq) {
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = (i < 4 ? s0[i] : s1[i - 4]) * scale;
    if (tok0 + MT2 > t1) {
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = tok0 + (i < 4 ? 0 : 16) + 4 * lq + (i & 3) < t1 ? v[i] : -INFINITY;
    }
  }
  // the block's maximum and the reference
  __device__ __forceinline__ void reference(float& m_run) {
    float bm = v[0];
#pragma unroll
    for (int i = 1; i < 8; ++i) bm = fmaxf(bm, v[i]);
    bm = ml_max4(bm);
    // bm is finite (every block has a token); the first block always raises
    raise = bm > m_run + kRescaleGap;
    const float m_new = raise ? bm : m_run;
    alpha = raise ? __expf(m_run - m_new) : 1.f;
    m_run = m_new;
    ps = 0.f;
  }
  // probability i
  __device__ __forceinline__ void prob(int i, float m_run) {
    const float e = __expf(v[i] - m_run);
    ps += e;
    pb[i] = (__bf16)e;
  }
  __device__ __forceinline__ void sum(float& l_part) { l_part = l_part * alpha + ps; }
};

// The 16 query rows of head block hb (rows past H_q read as zero).
__device__ __forceinline__ void mla_load_q(const MlaParams& p, int b, int hb, int lr, int lq, bf16x8 (&qf)[MSTEPS]) {
  const int h0 = hb * 16;
  const __amdgpu_buffer_rsrc_t rq =
      ml_rsrc(p.q + ((size_t)b * p.Hq + h0) * MD, (uint32_t)min(16, p.Hq - h0) * MD * 2u);
#pragma unroll
  for (int c = 0; c < MSTEPS; ++c)
    qf[c] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(
                                           rq, (uint32_t)(lr * MD + 32 * c + 8 * lq) * 2u, 0, 0));
}

// A task's unnormalised output, max and sum; lane (lr, lq) holds
// O^T[16 j + 4 lq + i][head 16 hb + lr].
__device__ __forceinline__ void mla_store(const MlaParams& p, int b, int split, int hb, int lr, int lq,
                                          const f32x4 (&o)[MV / 16], float m_run, float l_part) {
  l_part += __shfl_xor(l_part, 16);  // the four token groups of a head's sum
  l_part += __shfl_xor(l_part, 32);
  const int h = hb * 16 + lr;
  if (h < p.Hq) {
    const size_t row = ((size_t)b * p.Hq + h) * p.n_splits + split;
    float* dst = p.part_o + row * MV + 4 * lq;
#pragma unroll
    for (int j = 0; j < MV / 16; ++j) *reinterpret_cast<f32x4*>(dst + 16 * j) = o[j];
    if (lq == 0) {
      p.part_ml[row * 2] = m_run;
      p.part_ml[row * 2 + 1] = l_part;
    }
  }
}

// ---- wave form: one (request, split, head block) per wave ---------------
__device__ void mla_task(const MlaParams& p, int b, int split, int hb, unsigned char* __restrict__ vt) {
  const int lane = threadIdx.x & 63;
  const int lr = lane & 15, lq = lane >> 4;
  const int t0 = split * p.split;
  const int t1 = min(p.S, t0 + p.split);
  const int nblk = (t1 - t0 + MT - 1) / MT;
  const __amdgpu_buffer_rsrc_t rk = ml_rsrc(p.kv + (size_t)b * p.S * MD, (uint32_t)p.S * MD * 2u);
  bf16x8 qf[MSTEPS];
  mla_load_q(p, b, hb, lr, lq, qf);
  f32x4 o[MV / 16];
#pragma unroll
  for (int j = 0; j < MV / 16; ++j) o[j] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_part = 0.f;

  // key fragments of a block (16 tokens): step c holds values 32 c .. 32 c + 31
  bf16x8 kf[MSTEPS];
  auto load_block = [&](int blk) {
    const int tok = t0 + blk * MT + lr;
    const uint32_t base = tok < t1 ? (uint32_t)(tok * MD + 8 * lq) * 2u : kMlOOB;
#pragma unroll
    for (int c = 0; c < MSTEPS; ++c)
      kf[c] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rk, base, 64 * c, 0));
  };
  load_block(0);
  for (int blk = 0; blk < nblk; ++blk) {
    const f32x4 s = mla_scores(kf, qf);
    // the latent values of the block into the tile as they are (row: token,
    // 16 contiguous bytes per lane and step); this wave's reads of the
    // previous block are complete (its LDS accesses run in order)
#pragma unroll
    for (int c = 0; c < VSTEPS; ++c)
      *reinterpret_cast<v4u*>(vt + (uint32_t)lr * V_ROW + (uint32_t)(32 * c + 8 * lq) * 2u) =
          __builtin_bit_cast(v4u, kf[c]);
    // the next block's rows go out now (the fragments are consumed)
    if (blk + 1 < nblk) load_block(blk + 1);
    const i16x4 pb = mla_softmax(s, t0 + blk * MT, t1, p.scale, lq, o, m_run, l_part);
    wave_sync();  // the tile writes of every lane before any lane reads
    mla_pv(vt, V_ROW, pb, lr, lq, o);
    wave_sync();  // every lane's reads of the tile before the next block's writes
  }
  mla_store(p, b, split, hb, lr, lq, o, m_run, l_part);
}

// ---- workgroup forms: one (request, split, group of 4 NH head blocks) per
// workgroup, NH (1 or 2) head blocks per wave.  The rows go from memory
// straight into four shared LDS tiles of 32 tokens (buffer_load ... lds, two
// blocks ahead).  Every key fragment read from a tile feeds the score chains of
// the wave's NH head blocks and every joined value fragment their P.V products,
// so the 128-head form (NH = 2) reads half the LDS bytes per head of the
// 64-head form (NH = 1).  The output accumulators (128 per head block) stay in
// AGPRs (inline-asm MFMAs, with the wait states around their VALU accesses
// padded explicitly).  The softmax runs once per 32 tokens and P.V takes
// 32-deep products, so these forms round differently from the wave form
// (16-token blocks); per head both do the same operations in the same order,
// so their bits are the same, and none depends on the placement.
//
// What bounds it: one wave per SIMD (NH = 2 fills its registers), so nothing
// but the wave's own instruction stream can cover a read's or the softmax's
// latency.  The block's P.V is therefore split around the next block's scores
// and softmax (see below).  Whole calls, before (scores, softmax and P.V in
// turn; NH = 1 staged its rows in registers) and now, us: NH = 2, B=64, S=32768
// 660 and 608; B=16, S=8192, 512-token splits 64.2 and 59.0 (about 20 us of it
// do not depend on the tokens: the launch, the queries and 67 MB of fp32
// partials, which the merge reads in another 13); NH = 1, B=16, S=4096 47.3 and
// 36.7, B=1, S=32768 34.0 and 28.3.  Where the products and reads are placed
// (VA = 4 to 16, three or four tiles ahead) makes less than 1%.

// buffer descriptor words (uniform) for the asm loads
__device__ __forceinline__ i32x4 ml_rsrc_words(const void* base, uint32_t bytes) {
  const unsigned long long a = (unsigned long long)base;
  return i32x4{(int)__builtin_amdgcn_readfirstlane((uint32_t)a), (int)__builtin_amdgcn_readfirstlane((uint32_t)(a >> 32)),
               (int)__builtin_amdgcn_readfirstlane(bytes), 0x00020000};
}

// 16 bytes per lane from memory (byte offset voff + soff of the buffer) into
// LDS: lane L's bytes land at lds + 16 L.  The compiler does not see these
// loads; their completion is waited for explicitly (ml_vmwait) before the
// barrier that publishes the tile.
template <bool NT>  // non-temporal
__device__ __forceinline__ void ml_dma16(uint32_t lds, i32x4 rs, uint32_t voff, uint32_t soff) {
  if constexpr (NT)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen nt lds"
                 : : "s"(lds), "v"(voff), "s"(rs), "s"(soff) : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
               : : "s"(lds), "v"(voff), "s"(rs), "s"(soff) : "memory", "m0");
}
template <int N>
__device__ __forceinline__ void ml_vmwait() {
  asm volatile("s_waitcnt vmcnt(%0)" : : "i"(N) : "memory");
}

// acc += a . b with the accumulator in AGPRs
__device__ __forceinline__ void ml_mfma_acc(f32x4& acc, const bf16x8& a, const bf16x8& b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}
// wait states between the asm MFMAs and vector accesses of their accumulators
// (covers the longest dependency of the 16x16x32 shape)
__device__ __forceinline__ void ml_mfma_fence() {
  asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" ::: "memory");
}
// the accumulators materialised in AGPRs at this point of the program
template <int NH>
__device__ __forceinline__ void ml_pin(f32x4 (&o)[NH][MV / 16]) {
#pragma unroll
  for (int h = 0; h < NH; ++h)
#pragma unroll
    for (int j = 0; j < MV / 16; ++j) asm volatile("" : "+a"(o[h][j]));
}

template <int NH, bool ONCE>
__device__ void mla_wg_task(const MlaParams& p, int b, int split, int hg, unsigned char* __restrict__ tiles) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int lr = lane & 15, lq = lane >> 4;
  const int t0 = split * p.split;
  const int t1 = min(p.S, t0 + p.split);
  const int nblk = (t1 - t0 + MT2 - 1) / MT2;
  const int hb0 = (hg * MG + wave) * NH;
  // the request's rows; a split is a multiple of 32 tokens, so only the
  // request's last block is partial and its rows past S_k read as zero
  const i32x4 rk = ml_rsrc_words(p.kv + (size_t)b * p.S * MD, (uint32_t)p.S * MD * 2u);
  bf16x8 qf[NH][MSTEPS];
#pragma unroll
  for (int h = 0; h < NH; ++h) mla_load_q(p, b, hb0 + h, lr, lq, qf[h]);
  f32x4 o[NH][MV / 16];
#pragma unroll
  for (int h = 0; h < NH; ++h)
#pragma unroll
    for (int j = 0; j < MV / 16; ++j) o[h][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  ml_pin<NH>(o);
  ml_mfma_fence();
  float m_run[NH], l_part[NH];
#pragma unroll
  for (int h = 0; h < NH; ++h) {
    m_run[h] = -INFINITY;
    l_part[h] = 0.f;
  }

  // A tile is 9 pieces of 32 rows x 128 bytes; a row's 16-byte chunk c of a
  // piece lies at chunk c ^ ((row >> 1) & 7), which spreads both the 16 rows of
  // a key fragment and the 16 half-chunks of a transposing read over the
  // banks.  Load g of this wave fetches piece g of rows 8 w .. 8 w + 7, eight
  // lanes per whole 128-byte line.
  const int drow = 8 * wave + (lane >> 3);
  const uint32_t voff = (uint32_t)(drow * MD * 2 + ((lane & 7) ^ ((drow >> 1) & 7)) * 16);
  const uint32_t lds_base = (uint32_t)(size_t)tiles;  // a shared address's low word is its LDS address
  auto tile_at = [&](int blk) { return (uint32_t)__builtin_amdgcn_readfirstlane((blk % T2_TILES) * T2_BYTES); };
  // (a block past the last is loaded from an empty buffer: zeros, no traffic)
  auto dma = [&](int blk, int g) {
    i32x4 rs = rk;
    rs[2] = __builtin_amdgcn_readfirstlane(blk < nblk ? rk[2] : 0);
    const uint32_t so = (uint32_t)__builtin_amdgcn_readfirstlane((t0 + blk * MT2) * (MD * 2) + g * 128);
    ml_dma16<ONCE>(lds_base + tile_at(blk) + (uint32_t)(g * T2_GROUP_BYTES + wave * 1024), rs, voff, so);
  };
  // key fragment of step c, rows 16 half + lr: chunk 4 (c & 1) + lq of piece c / 2
  const uint32_t kb0 = (uint32_t)(lr * 128 + (lq ^ ((lr >> 1) & 7)) * 16);
  auto kread = [&](uint32_t tile, int c, bf16x8 (&k)[2]) {
    lds_u8* at = reinterpret_cast<lds_u8*>((size_t)(tile + (c & 1 ? kb0 ^ 64u : kb0)));
#pragma unroll
    for (int half = 0; half < 2; ++half)
      k[half] = *reinterpret_cast<lds_bf16x8*>(at + (c >> 1) * T2_GROUP_BYTES + half * 2048);
  };
  // value tile j (16 values), both 16-row halves: 8 bytes of rows 4 lq + lr / 4
  // in chunk 2 (j & 3) + (lr & 3) / 2 of piece j / 4
  const int trow = 4 * lq + (lr >> 2);
  const uint32_t tb0 = (uint32_t)(trow * 128 + (((lr >> 1) & 1) ^ ((trow >> 1) & 7)) * 16 + 8 * (lr & 1));
  auto tread = [&](uint32_t tile, int j, i16x4 (&v)[2]) {
    lds_u8* at = reinterpret_cast<lds_u8*>((size_t)(tile + (tb0 ^ (uint32_t)(32 * (j & 3)))));
#pragma unroll
    for (int half = 0; half < 2; ++half)
      v[half] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
          reinterpret_cast<lds_i16x4*>(at + (j >> 2) * T2_GROUP_BYTES + half * 2048));
  };
  // Two streams of MFMAs that need nothing of each other: the scores of block
  // blk + 1 (18 steps of NH head blocks x two 16-row halves) and the P.V of
  // block blk (32 value tiles x NH head blocks).  The first VA tiles go between
  // the score steps; the rest go with the softmax of block blk + 1, whose
  // vector instructions run while the matrix cores work on them.  Each stream's
  // reads are issued two steps or three tiles ahead.
  constexpr int VT = MV / 16, VA = 8, TD = 4;
  f32x4 sc[NH][2];
  bf16x8 pb[NH];  // block blk's probabilities
  Softmax32 sm[NH];
  bf16x8 kf[3][2];
  i16x4 ab[TD][2];
  auto pv_start = [&](uint32_t tile) {
#pragma unroll
    for (int j = 0; j < TD - 1; ++j) tread(tile, j, ab[j]);
  };
  auto pv = [&](uint32_t tile, int j) {
    i16x4 (&v)[2] = ab[j % TD];
    asm volatile("" : "+v"(v[0]), "+v"(v[1]));
    if (j + TD - 1 < VT) tread(tile, j + TD - 1, ab[(j + TD - 1) % TD]);
    const bf16x8 a = __builtin_bit_cast(bf16x8, __builtin_shufflevector(v[0], v[1], 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
    for (int h = 0; h < NH; ++h) ml_mfma_acc(o[h][j], a, pb[h]);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto score_start = [&](uint32_t tile) {
    kread(tile, 0, kf[0]);
    kread(tile, 1, kf[1]);
#pragma unroll
    for (int h = 0; h < NH; ++h) sc[h][0] = sc[h][1] = f32x4{0.f, 0.f, 0.f, 0.f};
  };
  // (with one row load of block lblk in every other step)
  auto score = [&](uint32_t tile, int i, int lblk) {
    bf16x8 (&k)[2] = kf[i % 3];
    asm volatile("" : "+v"(k[0]), "+v"(k[1]));
    if (i + 2 < MSTEPS) kread(tile, i + 2, kf[(i + 2) % 3]);
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int h = 0; h < NH; ++h)
        sc[h][u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k[u], qf[h][i], sc[h][u], 0, 0, 0);
    if ((i & 1) == 0) dma(lblk, i >> 1);
    __builtin_amdgcn_sched_barrier(0);
  };
  // piece x of a block's softmax
  constexpr int PIECES = 6 * NH;
  static_assert(VA <= MSTEPS && PIECES <= VT - VA, "at most one tile or piece per step");
  auto softmax = [&](int blk, int x) {
    const int h = x / 6, y = x % 6;
    if (y == 0)
      sm[h].scores(sc[h][0], sc[h][1], t0 + blk * MT2, t1, p.scale, lq);
    else if (y == 1)
      sm[h].reference(m_run[h]);
    else {
      sm[h].prob(2 * y - 4, m_run[h]);
      sm[h].prob(2 * y - 3, m_run[h]);
      if (y == 5) sm[h].sum(l_part[h]);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  static_assert(T2_GROUPS * 2 == MSTEPS, "one row load per two score steps");
  // block blk + 1 has landed (the loads of block blk + 2 may still be in
  // flight), and every wave is past block blk - 1, whose tile block blk + 3
  // takes; the output takes the factor of block blk before its P.V
  auto publish_and_rescale = [&](bool first) {
    ml_vmwait<T2_GROUPS>();
    __syncthreads();
    bool raise = false;
#pragma unroll
    for (int h = 0; h < NH; ++h) {
      pb[h] = sm[h].pb;
      raise = raise || sm[h].raise;
    }
    // (the first block raises every reference, but the output is still zero)
    if (!first && __ballot(raise)) {
      ml_mfma_fence();
      // one accumulator at a time through 4 VGPRs: each read is ordered
      // after the previous write-back by the empty asms
#pragma unroll
      for (int h = 0; h < NH; ++h)
#pragma unroll
        for (int j = 0; j < VT; ++j) {
          asm volatile("" : "+a"(o[h][j]));
          f32x4 t = o[h][j];
          asm volatile("" : "+v"(t));
          t *= sm[h].alpha;
          o[h][j] = t;
          asm volatile("" : "+a"(o[h][j]));
        }
      ml_mfma_fence();
    }
  };
  // blocks 0 and 1 in flight, the scores of block 0 (with block 2's loads)
#pragma unroll
  for (int g = 0; g < T2_GROUPS; ++g) dma(0, g);
#pragma unroll
  for (int g = 0; g < T2_GROUPS; ++g) dma(1, g);
  ml_vmwait<T2_GROUPS>();
  __syncthreads();
  score_start(lds_base);
#pragma unroll
  for (int i = 0; i < MSTEPS; ++i) score(lds_base, i, 2);
#pragma unroll
  for (int x = 0; x < PIECES; ++x) softmax(0, x);
  int blk = 0;
  for (; blk + 1 < nblk; ++blk) {
    publish_and_rescale(blk == 0);
    const uint32_t vt = lds_base + tile_at(blk), st = lds_base + tile_at(blk + 1);
    pv_start(vt);
    score_start(st);
#pragma unroll
    for (int i = 0; i < MSTEPS; ++i) {
      score(st, i, blk + 3);
      if ((i + 1) * VA / MSTEPS > i * VA / MSTEPS) pv(vt, i * VA / MSTEPS);
    }
#pragma unroll
    for (int j = VA; j < VT; ++j) {
      pv(vt, j);
      const int x = (j - VA) * PIECES / (VT - VA);
      if ((j - VA + 1) * PIECES / (VT - VA) > x) softmax(blk + 1, x);
    }
  }
  publish_and_rescale(blk == 0);
  pv_start(lds_base + tile_at(blk));
#pragma unroll
  for (int j = 0; j < VT; ++j) pv(lds_base + tile_at(blk), j);
  ml_vmwait<0>();  // the last zero fills
  // (the next task's first loads overwrite tiles other waves may still read)
  __syncthreads();
  ml_mfma_fence();
#pragma unroll
  for (int h = 0; h < NH; ++h) mla_store(p, b, split, hb0 + h, lr, lq, o[h], m_run[h], l_part[h]);
}

__global__ void __launch_bounds__(64 * MW) mla_decode_split(MlaParams p) {
  __shared__ __attribute__((aligned(16))) unsigned char vt_all[MW][V_BYTES];
  __shared__ int box[2];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const bool aware = p.quota_off != nullptr;
  int own = 0;
  if (aware) {
    uint32_t xr;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xr));
    own = (int)(xr & 0xFu);
    if (own >= p.n_x || !((p.allow >> own) & 1u)) return;  // an XCD outside the set
  }
  // Oblivious: one group of 4 tasks, workgroup i's.  Aware: claims, own share
  // first, then the others in turn; wave 0 reads every counter in one round
  // trip and only adds to shares that still have groups; the loop ends when
  // each counter has passed its share.  One call site of the task body.
  for (int round = 0;; ++round) {
    int base, end;
    if (!aware) {
      if (round > 0) break;
      base = blockIdx.x * MW;
      end = p.tasks;
    } else {
      if (wave == 0) {
        int rem = 0, y = 0, b0 = 0, b1 = 0;
        if (lane < p.n_x) {
          y = (own + lane) % p.n_x;
          b0 = p.quota_off[y];
          b1 = p.quota_off[y + 1];
          const int taken =
              __hip_atomic_load(&p.claim[y * kMlClaimStride], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          rem = (b1 - b0 + MW - 1) / MW - taken;
        }
        unsigned long long open = __ballot(lane < p.n_x && rem > 0);
        int got_base = -1, got_end = 0;
        while (open && got_base < 0) {
          const int l = __builtin_ctzll(open);
          open &= open - 1;
          int got = -1;
          if (lane == l) {
            const int g = atomicAdd(&p.claim[y * kMlClaimStride], 1);
            if (b0 + g * MW < b1) got = b0 + g * MW;
          }
          got = __shfl(got, l);
          if (got >= 0) {
            got_base = got;
            got_end = __shfl(b1, l);
          }
        }
        if (lane == 0) {
          box[0] = got_base;
          box[1] = got_end;
        }
      }
      __syncthreads();
      base = box[0];
      end = box[1];
      __syncthreads();
      if (base < 0) break;
    }
    if (base + wave < end) {
      int b, split, hb;
      mla_task_of(p, aware, base + wave, b, split, hb);
      mla_task(p, b, split, hb, vt_all[wave]);
    }
  }
}

// Workgroup form: tasks (request, split, group of 4 head blocks), numbered
// with the group fastest (aware) or group major (oblivious).  Oblivious: task
// i on workgroup i.  Aware: claims of one task, own share first, then the
// others, as in the wave form.
// KIND 1, 2: that many head blocks per wave; 3, 4: the same with the rows loaded
// non-temporally.
template <int KIND>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) mla_decode_split_wg(MlaParams p) {
  __shared__ __attribute__((aligned(1024))) unsigned char tiles[T2_TILES * T2_BYTES];
  __shared__ int box[1];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const bool aware = p.quota_off != nullptr;
  constexpr int NH = KIND > 2 ? KIND - 2 : KIND;
  const int groups = p.hblocks / (MG * NH);
  int own = 0;
  if (aware) {
    uint32_t xr;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xr));
    own = (int)(xr & 0xFu);
    if (own >= p.n_x || !((p.allow >> own) & 1u)) return;  // an XCD outside the set
  }
  for (int round = 0;; ++round) {
    int task;
    if (!aware) {
      if (round > 0 || (int)blockIdx.x >= p.tasks) break;
      task = blockIdx.x;
    } else {
      if (wave == 0) {
        int rem = 0, y = 0, b0 = 0, b1 = 0;
        if (lane < p.n_x) {
          y = (own + lane) % p.n_x;
          b0 = p.quota_off[y];
          b1 = p.quota_off[y + 1];
          const int taken =
              __hip_atomic_load(&p.claim[y * kMlClaimStride], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          rem = (b1 - b0) - taken;
        }
        unsigned long long open = __ballot(lane < p.n_x && rem > 0);
        int got_task = -1;
        while (open && got_task < 0) {
          const int l = __builtin_ctzll(open);
          open &= open - 1;
          int got = -1;
          if (lane == l) {
            const int g = atomicAdd(&p.claim[y * kMlClaimStride], 1);
            if (b0 + g < b1) got = b0 + g;
          }
          got_task = __shfl(got, l);
        }
        if (lane == 0) box[0] = got_task;
      }
      __syncthreads();
      task = box[0];
      __syncthreads();
      if (task < 0) break;
    }
    int b, split, hg;
    if (aware) {
      hg = task % groups;
      const int r = task / groups;
      split = r % p.n_splits;
      b = r / p.n_splits;
    } else {
      const int bs = p.B * p.n_splits;
      hg = task / bs;
      const int r = task - hg * bs;
      split = r % p.n_splits;
      b = r / p.n_splits;
    }
    mla_wg_task<NH, (KIND > 2)>(p, b, split, hg, tiles);
  }
}

// Merge of the splits of every (request, head) row (split_merge.h); also
// clears the aware form's claim counters (the split launch is complete).
template <int CH>
__global__ void __launch_bounds__(64 * kMergeWaves) mla_decode_merge(const float* __restrict__ part_o,
                                                                     const float* __restrict__ part_ml, int rows,
                                                                     int n_splits, int wpr, uint16_t* __restrict__ o,
                                                                     float* __restrict__ lse, int* claim,
                                                                     int n_claim) {
  if (claim && blockIdx.x == 0 && blockIdx.y == 0 && (int)threadIdx.x < n_claim) claim[threadIdx.x * kMlClaimStride] = 0;
  merge_split_rows<MV, CH>(part_o, part_ml, rows, n_splits, wpr, o, lse);
}

}  // namespace

int launch_mla_decode(const MlaLaunch& a, hipStream_t s) {
  MlaParams p;
  p.q = static_cast<const uint16_t*>(a.q);
  p.kv = static_cast<const uint16_t*>(a.kv);
  p.part_o = a.part_o;
  p.part_ml = a.part_ml;
  p.quota_off = a.d_quota_off;
  p.claim = a.d_claim;
  p.allow = a.allow;
  p.B = a.B;
  p.Hq = a.Hq;
  p.S = a.S;
  p.split = a.split;
  p.n_splits = a.n_splits;
  p.hblocks = (a.Hq + 15) / 16;
  if (a.form < 0 || a.form > 2) return fail(ASYM_EINVAL, "mla: unknown kernel form");
  const int per_task = mla_form_head_blocks(a.form);
  if (p.hblocks % per_task) return fail(ASYM_EINVAL, "mla: the head count does not suit the kernel form");
  p.tasks = a.B * a.n_splits * (p.hblocks / per_task);
  p.n_x = a.n_x;
  p.scale = a.scale;
  if (a.d_quota_off && (!a.d_claim || a.n_x > 64)) return fail(ASYM_EINVAL, "mla: aware launch without claim counters");
  if (a.grid < 1) return fail(ASYM_EINVAL, "mla: empty grid");
  // Where one workgroup reads a row for all its heads, rows that exceed the
  // memory-side cache (256 MiB) are loaded non-temporally; smaller caches may
  // still be resident, and several groups of heads share a row's second read.
  // Measured, caches of four calls in turn, us, ordinary loads first: 128 heads,
  // 151 MB 63.3 and 63.5 (resident 59.1 and 63.5), 604 MB 196 and 187, 2.4 GB
  // 607 and 594; 64 heads, 604 MB 149 and 138.  The wave form's loads lose
  // everywhere (16 heads, 604 MB 123 and 126).
  const bool once = p.hblocks == per_task && (int64_t)a.B * a.S * MD * 2 >= (256ll << 20);
  if (a.form != 0) {
    auto split_wg = a.form == 2 ? (once ? mla_decode_split_wg<4> : mla_decode_split_wg<2>)
                                : (once ? mla_decode_split_wg<3> : mla_decode_split_wg<1>);
    hipLaunchKernelGGL(split_wg, dim3((unsigned)a.grid), dim3(256), 0, s, p);
  } else
    hipLaunchKernelGGL(mla_decode_split, dim3((unsigned)a.grid), dim3(64 * MW), 0, s, p);
  ASYM_HIP(hipGetLastError());
  const int rows = a.B * a.Hq;
  const int wpr = merge_waves_per_row(a.n_splits), rows_per_wg = kMergeWaves / wpr;
  const int groups = (rows + rows_per_wg - 1) / rows_per_wg;
  const int ch = merge_column_chunks(groups, MV / 64);
  auto merge = ch == 8 ? mla_decode_merge<8> : ch == 4 ? mla_decode_merge<4> : ch == 2 ? mla_decode_merge<2>
                                                                                      : mla_decode_merge<1>;
  hipLaunchKernelGGL(merge, dim3((unsigned)groups, (unsigned)ch), dim3(64 * kMergeWaves), 0, s, a.part_o, a.part_ml,
                     rows, a.n_splits, wpr, static_cast<uint16_t*>(a.o), a.lse, a.d_quota_off ? a.d_claim : nullptr,
                     a.n_x);
  ASYM_HIP(hipGetLastError());
  return ASYM_OK;
}

int mla_tasks_per_workgroup() { return MW; }

int mla_form_head_blocks(int form) { return form ? MG * form : 1; }

}  // namespace asym
