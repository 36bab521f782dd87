// Causal GQA prefill attention on bf16 MFMA (gfx950), block-sparse over the
// selected key blocks (Section 4.2, Appendix A Eq. t_spa) or dense (the
// full-attention baseline).
//
// One workgroup = one 128-row query tile of one (batch, query head); four
// waves own 32 query rows each.  Keys are visited in 64-key sub-blocks copied
// straight from global memory into a two-stage LDS ring (no register
// staging); per sub-block each wave computes
//   S^T = K Q^T        2 x 8  MFMA 32x32x16 (keys on M, queries on N)
//   online softmax     fp32, base 2, the row of one query lives in one lane
//                      pair (lanes l and l^32)
//   O^T += V^T P^T     4 x 4  MFMA 32x32x16 (head dims on M)
// With keys on the M dimension every lane owns one query's scores, so the
// softmax needs a single cross-lane exchange per sub-block, and the output
// rescale uses the lane's own running maximum.
//
// MFMA 32x32x16 bf16 operand layout (lane l, half h = l / 32):
//   A[i][k]: lane holds i = l % 32, k = 8h .. 8h+7
//   B[k][j]: lane holds j = l % 32, k = 8h .. 8h+7
//   D[i][j]: lane holds j = l % 32, i = 8 (r / 4) + 4h + r % 4, r = 0..15
// The keys of the S^T output a lane holds are therefore not contiguous; the
// V^T operand is read from the row-major V tile with the transposing LDS read
// (ds_read_b64_tr_b16) in that same key order, so P^T feeds the second
// product straight from registers.
//
// Dense workgroups are mapped so that each XCD (dispatched round-robin)
// receives a contiguous run of (batch, KV head, tile, query head) work: the G
// query heads that share a K/V head, and neighbouring tiles, run on one XCD
// and reuse K/V blocks from its L2.  Heavier (later) tiles are issued first.
//
// Sparse work per head is uneven (budgets differ per head, up to 3x).  With a
// scheduling workspace the sparse kernel is persistent: two workgroups per
// CU, each taking (tile, KV group, query head) items from a queue of its own
// XCD (the XCD's KV groups, or its share of one group's tiles in runs of
// kRun, heaviest tiles first) through an atomic counter, and from the other
// XCDs' queues once its own is empty.  Each XCD's L2 then holds the K/V of
// its own groups, whose tiles select largely the same blocks, and the
// stealing evens out the groups' different loads.  Without a workspace (or
// for KV-group counts that do not tile the XCDs) the grid is static: the KV
// groups rotate over the XCDs every 4 tiles, heaviest tiles first.
//
// Launches of few tiles (attn_split_kernel; the rule is at split_tiles) split
// each tile's keys over the waves instead, dense and sparse alike.
#include "ei_internal.h"

#include <math.h>

namespace ei {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

constexpr int kThreads = 256;
constexpr int kTileQ = 128;
constexpr int kSub = 64;            // keys per staged sub-block
constexpr int kXcds = 8;
static_assert(kXcds == kSchedCounters, "one queue counter per XCD");
constexpr unsigned kRotRun = 4;    // tiles a KV group stays on one XCD (static sparse grid)
constexpr unsigned kRun = 16;      // tile run per XCD when XCDs share a KV group (persistent)
// Where no item has more than kShortItem steps (the list's capacity), each
// draws the next item's ticket while it runs: the atomic's round trip, ~1 us of
// an item's ~20, is hidden (budgets of 256 tokens, 128-key blocks: 16 heads x
// 10240 tokens 88.9 -> 83.3 us, x 7808 80.1 -> 75.3).  With longer items about,
// a ticket drawn early keeps its tile waiting at the end of the launch while
// other workgroups run dry (4k tokens 0.96x; drawn by items of any length
// 0.89x).
constexpr int kShortItem = 16;
constexpr unsigned kHeadRun = 16;  // tiles of one query head in a row in an XCD's queue

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 w) { return __builtin_bit_cast(bf16x8, w); }

// Two fp32 values -> packed bf16 pair (round to nearest even), one instruction.
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  const f32x2 x = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(x, bf16x2));
}

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4_t;

// One LDS stage holds a 64-key sub-block of K and of V, each row-major with
// 256-byte rows whose 16-byte chunks are XOR-swizzled per row.  K rows are
// read 16 at a time at one logical chunk, so K uses chunk ^ (r % 16).  The
// transposing V reads take, per 16 lanes, the same 32-byte chunk pair of 4
// consecutive rows (and per 32 lanes a 64-byte chunk quad), so V uses
// chunk ^ h(r % 4) with h = {0, 6, 12, 10}: the pair index and the quad index
// then differ across any 4 consecutive rows and every read is free of bank
// conflicts.
constexpr int kRowBytes = kHeadDim * 2;
constexpr int kTileBytes = kSub * kRowBytes;       // 16 KiB
constexpr int kStageBytes = 2 * kTileBytes;        // K then V

__device__ __forceinline__ int swz(int row, int chunk) { return chunk ^ (row & 15); }
__device__ __forceinline__ int swz_v(int row, int chunk) {
  return chunk ^ ((0xAC60 >> (4 * (row & 3))) & 15);
}

// NC copies of 16 bytes per lane from global memory straight into LDS
// (global_load_lds_dwordx4: lane l's bytes land at M0 + 16 l), from a
// wave-uniform base (SGPR pair) and 32-bit lane offsets, each 1 KB further on
// than the last in memory and in LDS: the instruction's offset moves both
// addresses, so M0 is set once.  Written as asm so that the compiler does not
// treat a copy as a pending LDS write before every later LDS read: completion
// is enforced explicitly with a vmcnt wait before the barrier that publishes a
// stage.
template <int NC>
__device__ __forceinline__ void copy_rows_to_lds(const unsigned char* sbase, const uint32_t* off,
                                                 uint32_t lds_base) {
  static_assert(NC == 2 || NC == 4, "copies of a wave per stage and tensor");
  if constexpr (NC == 4)
    asm volatile(
        "s_mov_b32 m0, %0\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %1, %5\n\t"
        "global_load_lds_dwordx4 %2, %5 offset:1024\n\t"
        "global_load_lds_dwordx4 %3, %5 offset:2048\n\t"
        "global_load_lds_dwordx4 %4, %5 offset:3072"
        :
        : "s"(lds_base), "v"(off[0]), "v"(off[1]), "v"(off[2]), "v"(off[3]), "s"(sbase)
        : "memory", "m0");
  else
    asm volatile(
        "s_mov_b32 m0, %0\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %1, %3\n\t"
        "global_load_lds_dwordx4 %2, %3 offset:1024"
        :
        : "s"(lds_base), "v"(off[0]), "v"(off[1]), "s"(sbase)
        : "memory", "m0");
}

// One such copy.
__device__ __forceinline__ void copy_row_to_lds(const unsigned char* sbase, uint32_t off,
                                                uint32_t lds_base) {
  asm volatile(
      "s_mov_b32 m0, %0\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %1, %2"
      :
      : "s"(lds_base), "v"(off), "s"(sbase)
      : "memory", "m0");
}

// Global -> LDS without registers: each of 16 / NC waves moves 4 NC rows of K
// and of V (NC + NC instructions of 64 lanes x 16 bytes).  Lane L of
// instruction j fills row 4 NC w + 4 j + L / 16, swizzled chunk position
// L % 16.  koff holds those K rows' byte offsets inside a block less the
// 1024 j of the instruction's offset, voff the same for V (one value: its
// swizzle repeats every 4 rows).  Rows at or past N are read from row N - 1
// (finite data whose scores are masked).
template <int NC>
__device__ __forceinline__ void issue_stage(unsigned char* stage, const uint16_t* __restrict__ kh,
                                            const uint16_t* __restrict__ vh, int k0, int N,
                                            int wave, int lane, const uint32_t* koff,
                                            uint32_t voff) {
  const uint32_t dst = (uint32_t)(uintptr_t)stage +
                       (uint32_t)(4 * NC * __builtin_amdgcn_readfirstlane(wave) * kRowBytes);
  // (the second half of a last 128-key block may lie past the sequence's end)
  const int kc = min(k0, N - 1);
  const unsigned char* kb = (const unsigned char*)kh + (size_t)kc * kRowBytes;
  const unsigned char* vb = (const unsigned char*)vh + (size_t)kc * kRowBytes;
  if (k0 + kSub <= N) {   // whole block inside the sequence
    copy_rows_to_lds<NC>(kb, koff, dst);
    uint32_t vo[NC];
#pragma unroll
    for (int j = 0; j < NC; ++j) vo[j] = voff;
    copy_rows_to_lds<NC>(vb, vo, dst + kTileBytes);
    return;
  }
  // The block that holds the sequence's end.  (Opaque: its row offsets are
  // formed here, not kept across the loop.)
  asm volatile("" : "+v"(lane));
#pragma unroll
  for (int j = 0; j < NC; ++j) {
    const int row = 4 * NC * wave + 4 * j + (lane >> 4), pos = lane & 15;
    const uint32_t roff = (uint32_t)((min(k0 + row, N - 1) - kc) * kRowBytes);
    copy_row_to_lds(kb, roff + 16 * swz(row, pos), dst + 1024 * j);
    copy_row_to_lds(vb, roff + 16 * swz_v(row, pos), dst + 1024 * j + kTileBytes);
  }
}

template <int NC>
__device__ __forceinline__ void stage_offsets(int wave, int lane, uint32_t* koff, uint32_t& voff) {
  const int row = 4 * NC * wave + (lane >> 4);
#pragma unroll
  for (int j = 0; j < NC; ++j)
    koff[j] = (uint32_t)(row * kRowBytes + 16 * swz(row + 4 * j, lane & 15));
  voff = (uint32_t)(row * kRowBytes + 16 * swz_v(row, lane & 15));
}

// K operand of S^T = K Q^T: 8 bf16 of key row `row`, dims 16 s + 8 h .. +7.
__device__ __forceinline__ bf16x8 read_k(const unsigned char* stage, int row, int s, int h) {
  return as_bf16x8(*(const uint4*)(stage + row * kRowBytes + 16 * swz(row, 2 * s + h)));
}

// V^T operand of O^T += V^T P^T for head-dim tile dt and 16-key step t, read
// transposed from the row-major V tile: lane l (group g = l / 16, i = l % 16)
// receives V[key][32 dt + 16 (g % 2) + i] for the keys 16 t + 8 a + 4 (g / 2)
// + 0..3, a = 0, 1 -- the key order of the S^T output.
__device__ __forceinline__ bf16x8 read_vt(const unsigned char* stage, int dt, int t, int lane) {
  const int g = lane >> 4, i = lane & 15;
  const int d = 32 * dt + 16 * (g & 1) + 4 * (i & 3);
  const unsigned char* vt = stage + kTileBytes;
  s16x4 r[2];
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    const int row = 16 * t + 8 * a + 4 * (g >> 1) + (i >> 2);
    const unsigned char* p = vt + row * kRowBytes + 16 * swz_v(row, d >> 3) + 2 * (d & 7);
    r[a] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)p);
  }
  const uint2 lo = __builtin_bit_cast(uint2, r[0]), hi = __builtin_bit_cast(uint2, r[1]);
  return as_bf16x8(make_uint4(lo.x, lo.y, hi.x, hi.y));
}

// Wait until at most n vector-memory operations of this wave are in flight
// (gfx9 encoding: vmcnt in bits 3:0 and 15:14; expcnt, lgkmcnt left at max).
#define EI_WAIT_VMCNT(n) \
  __builtin_amdgcn_s_waitcnt(((n) & 15) | (((n) >> 4) << 14) | (7 << 4) | (15 << 8))

// Wait until every LDS read of this wave has returned (lgkmcnt 0, others max).
#define EI_WAIT_LGKM0() __builtin_amdgcn_s_waitcnt(15 | (3 << 14) | (7 << 4))

// The persistent sparse schedule (see the file comment).  S = 1: XCD x owns
// the KV groups x, x + 8, ... (ngx of them), its queue running over chunks of
// kHeadRun tile ranks (heaviest first) and, inside a chunk, over its (group,
// query head) pairs, each taking the chunk's tiles in a row (at the 128k
// layer: 10.5 GB fetched per launch against 13.7 GB with the heads of a
// tile next to each other, and equal or 1-2% faster).  S > 1 (8 = S x the
// number of groups): XCD x owns group x % NG and, of its tiles ranked
// heaviest first, the runs of kRun ranks with (rank / kRun) % S == x / NG.
// per_x[x] is the length of XCD x's queue.  Every item appears in exactly
// one queue.
struct XcdPlan {
  unsigned S, ngx, per_x[kXcds];
};

// Item idx of XCD x's queue -> (tile, query head in the group, KV group).
__device__ __forceinline__ void plan_item(const XcdPlan& pl, unsigned x, unsigned idx, int n_tiles,
                                          unsigned G, unsigned NG, int& tile, int& hh,
                                          unsigned& bg) {
  unsigned tr;
  if (pl.S == 1) {
    // chunks of kHeadRun tile ranks, heaviest first; inside a chunk the
    // (group, head) pairs in turn, each over the chunk's ranks
    const unsigned per_rank = G * pl.ngx;
    const unsigned c = idx / (kHeadRun * per_rank), j = idx % (kHeadRun * per_rank);
    const unsigned rr = min(kHeadRun, (unsigned)n_tiles - c * kHeadRun);   // ranks in the chunk
    const unsigned hg = j / rr;
    tr = c * kHeadRun + j % rr;
    hh = (int)(hg % G);
    bg = x + kXcds * (hg / G);
  } else {
    const unsigned kq = idx / G, part = x / NG;
    hh = (int)(idx % G);
    bg = x % NG;
    tr = (kq / kRun) * (pl.S * kRun) + part * kRun + kq % kRun;
  }
  tile = n_tiles - 1 - (int)tr;
}

// Queue counters of one call (the caller's scheduling workspace), zeroed on
// the call's stream before the kernel reads them (in the one-call path by the
// probe's first kernel).
__global__ void sched_reset_kernel(uint32_t* __restrict__ sched) {
  if (threadIdx.x < kXcds) sched[threadIdx.x] = 0u;
}

// Lazy rescaling: the running maximum m is only raised when a new score
// exceeds it by more than 8 (base-2 units), so O and l are rescaled rarely; O
// and l always share the same reference, so the result is the exact softmax.
// A sub-block's probabilities are first formed against the current m without
// its row maximum: if every lane's sum of them stays <= 2^32 (so each
// probability does, and O, l stay far from overflow), they are kept.
// Otherwise (the first sub-block, a score more than 32 above m, or an
// overflow) the wave takes the row maxima, raises m by the rule above and
// forms them again.
constexpr float kRescaleThreshold = 8.0f;
constexpr float kFastLimit = 0x1p32f;

// Valid prefix of a block list of c entries, 64 at a time: strictly
// ascending, inside [0, C_B), and not wholly after the tile's last query.
template <int SUB>
__device__ __forceinline__ int valid_prefix(const int32_t* lst, int c, int CB, int q_last,
                                            int lane) {
  int nv = 0;
  for (int base = 0; base < c; base += kWave) {
    const int e = base + lane;
    bool ok = false;
    if (e < c) {
      const int blk = lst[e];
      const int prv = e > 0 ? lst[e - 1] : -1;
      ok = blk > prv && blk < CB && blk * SUB * kSub <= q_last;
    }
    const uint64_t bad = ~__builtin_amdgcn_ballot_w64(ok);
    if (bad != 0) {
      nv = base + (int)__builtin_ctzll(bad);
      break;
    }
    nv = base + kWave;
  }
  return min(nv, c);
}

// One 64-key sub-block (staged at st, first key k0) for the wave's 32 query
// rows: S^T = K Q^T, the causal / length mask, the online softmax with lazy
// rescaling, and O^T += V^T P^T.
// `scored` runs once the K operands have been read.  With LATE_V the V tile is
// read after the softmax only, behind `v_ready`.
struct Nothing {
  __device__ __forceinline__ void operator()() const {}
};
template <int MODE, bool LATE_V = false, class Scored = Nothing, class VReady = Nothing>
__device__ __forceinline__ void compute_step(const unsigned char* st, int k0, int qw0, int qrow,
                                             int N, int jq, int hf, int lane, const bf16x8* qf,
                                             float sc_log2, f32x16* oacc, float& m_i, float& l_i,
                                             Scored scored = {}, VReady v_ready = {}) {
  // S^T = K Q^T for the 64 keys (two 32-key tiles): every operand read is
  // issued before the first product, and the first V^T operands arrive during
  // the softmax.  Left to the scheduler, each product of the first key tile
  // waited for a read issued after the one before it (a read's latency is
  // longer than a product), and so did every second product of O^T.  What
  // remains is bound by power: the same launch on all-zero inputs runs 34%
  // faster (as a large matrix product does, 29%), so the earlier operands
  // shorten dense 16384 x 32 heads by 7% on zeros and by 3.2% on real data
  // (1993 -> 1931 us, 1.14 PFLOP/s; a large matrix product: 1.36), the sparse
  // 128k layer, with the cheaper stage copies, by 3% (6210 -> 6032 us).
  f32x16 sacc[2];
  bf16x8 kf[2][8];
#pragma unroll
  for (int s = 0; s < 8; ++s)
#pragma unroll
    for (int u = 0; u < 2; ++u) kf[u][s] = read_k(st, 32 * u + jq, s, hf);
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int r = 0; r < 16; ++r) sacc[u][r] = 0.0f;
#pragma unroll
  for (int s = 0; s < 8; ++s)
#pragma unroll
    for (int u = 0; u < 2; ++u)
      sacc[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[u][s], qf[s], sacc[u], 0, 0, 0);
  __builtin_amdgcn_sched_group_barrier(0x100, 16, 0);   // 16 LDS reads
  __builtin_amdgcn_sched_group_barrier(0x008, 16, 0);   // 16 MFMAs
  scored();
  bf16x8 vf[2][4];
  if constexpr (!LATE_V) {
#pragma unroll
    for (int s = 0; s < 4; ++s) vf[0][s] = read_vt(st, 0, s, lane);
    asm volatile("" ::: "memory");   // (keeps these reads ahead of the softmax)
  }
  // mask keys after the query (causal) or at / past N; branch-free
  const bool need_mask = (MODE != kDenseFull && k0 + kSub - 1 > qw0) || (k0 + kSub > N);
  if (need_mask) {
    const int lim = (MODE == kDenseFull ? N - 1 : min(qrow, N - 1)) - k0 - 4 * hf;
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int kk = 32 * u + 8 * (r >> 2) + (r & 3);
        sacc[u][r] = (kk <= lim) ? sacc[u][r] : -INFINITY;
      }
  }
  uint4 pw[4];   // P^T as bf16, one 16-key MFMA step each
  float lsum;
  auto probs = [&](float mneg) {
    lsum = 0.0f;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int u = s >> 1, base = 8 * (s & 1);
      float p[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        p[e] = __builtin_amdgcn_exp2f(fmaf(sacc[u][base + e], sc_log2, mneg));
        lsum += p[e];
      }
      pw[s] = make_uint4(pack_bf16x2(p[0], p[1]), pack_bf16x2(p[2], p[3]),
                         pack_bf16x2(p[4], p[5]), pack_bf16x2(p[6], p[7]));
    }
  };
  bool kept = false;
  if (__builtin_amdgcn_ballot_w64(m_i == -INFINITY) == 0) {
    probs(-m_i);
    kept = __builtin_amdgcn_ballot_w64(!(lsum <= kFastLimit)) == 0;   // NaN fails too
  }
  if (!kept) {
    float mx = -INFINITY;
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sacc[u][r]);
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    const float mcand = mx * sc_log2;
    if (__builtin_amdgcn_ballot_w64(mcand > m_i + kRescaleThreshold) != 0) {
      const float m_new = fmaxf(m_i, mcand);
      const float alpha = (m_new == -INFINITY) ? 1.0f : __builtin_amdgcn_exp2f(m_i - m_new);
      l_i *= alpha;
#pragma unroll
      for (int d = 0; d < 4; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[d][r] *= alpha;
      m_i = m_new;
    }
    probs((m_i == -INFINITY) ? 0.0f : -m_i);
  }
  l_i += lsum;
  // O^T += V^T P^T, the operands of the next head-dim tile read ahead
  if constexpr (LATE_V) {
    v_ready();
#pragma unroll
    for (int s = 0; s < 4; ++s) vf[0][s] = read_vt(st, 0, s, lane);
  }
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    if (d < 3) {
#pragma unroll
      for (int s = 0; s < 4; ++s) vf[(d + 1) & 1][s] = read_vt(st, d + 1, s, lane);
    }
#pragma unroll
    for (int s = 0; s < 4; ++s)
      oacc[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[d & 1][s], as_bf16x8(pw[s]), oacc[d], 0,
                                                       0, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, 8, 1);
    __builtin_amdgcn_sched_group_barrier(0x008, 4, 1);
  }
}

// O = O^T / l for the lane's query row, bf16.
__device__ __forceinline__ void store_rows(uint16_t* __restrict__ o, size_t row_base, int hf,
                                           const f32x16* oacc, float l_i) {
  const float l = l_i + __shfl_xor(l_i, 32);
  const float inv = l > 0.0f ? 1.0f / l : 0.0f;
  uint16_t* op = o + row_base * kHeadDim;
#pragma unroll
  for (int d = 0; d < 4; ++d)
#pragma unroll
    for (int gq = 0; gq < 4; ++gq) {
      const int dim = 32 * d + 8 * gq + 4 * hf;
      *(uint2*)(op + dim) =
          make_uint2(pack_bf16x2(oacc[d][4 * gq] * inv, oacc[d][4 * gq + 1] * inv),
                     pack_bf16x2(oacc[d][4 * gq + 2] * inv, oacc[d][4 * gq + 3] * inv));
    }
}

template <int MODE, int SUB>
__global__ __launch_bounds__(kThreads, 2) void attn_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
    const uint16_t* __restrict__ v, uint16_t* __restrict__ o, int B, int Hq, int Hkv, int N,
    int n_tiles, int Ls, int CS, int CB, float sc_log2, const int32_t* __restrict__ bidx,
    const int32_t* __restrict__ bcnt, int kmax, uint32_t* __restrict__ sched,
    const XcdPlan plan) {
  // two LDS objects (not one array) so that the compiler can tell the copy
  // into one stage from the reads of the other
  __shared__ __attribute__((aligned(1024))) unsigned char stage0[kStageBytes];
  __shared__ __attribute__((aligned(1024))) unsigned char stage1[kStageBytes];
  __shared__ unsigned s_x, s_idx;   // the persistent workgroup's next item

  const unsigned G = (unsigned)(Hq / Hkv);
  const unsigned total = (unsigned)B * (unsigned)Hq * (unsigned)n_tiles;
  const bool pers = MODE == kSparse && sched != nullptr;
  // this workgroup's XCD (XCC_ID register): its own queue comes first
  const unsigned x0 = pers ? (__builtin_amdgcn_s_getreg((31 << 11) | 20) & (kXcds - 1)) : 0u;
  unsigned ticket = 0u;   // (thread 0)
  bool taken = false;
  for (;;) {
    int hh, tile, g, b;
    if (pers) {
      if (threadIdx.x == 0) {
        unsigned xs = kXcds, is = 0;
        for (unsigned d = 0; d < kXcds && xs == kXcds; ++d) {
          const unsigned x = (x0 + d) & (kXcds - 1);
          if (plan.per_x[x] == 0) continue;
          const unsigned t = d == 0 && taken ? ticket : atomicAdd(&sched[x], 1u);
          if (t < plan.per_x[x]) {
            xs = x;
            is = t;
          }
        }
        s_x = xs;
        s_idx = is;
      }
      taken = false;
      // (the previous item's closing barrier keeps this write after every
      // wave's read of the last item)
      __syncthreads();
      // (wave-uniform: everything derived from the item stays in scalar registers)
      const unsigned xs = __builtin_amdgcn_readfirstlane(s_x);
      if (xs == kXcds) return;   // every queue is empty
      unsigned bg;
      plan_item(plan, xs, __builtin_amdgcn_readfirstlane(s_idx), n_tiles, G, (unsigned)(B * Hkv), tile, hh, bg);
      b = (int)(bg / (unsigned)Hkv);
      g = (int)(bg % (unsigned)Hkv);
    } else if (MODE != kSparse) {
      const unsigned per_xcd = gridDim.x / kXcds;
      unsigned t = (blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;
      if (t >= total) return;
      hh = (int)(t % G);
      t /= G;
      tile = n_tiles - 1 - (int)(t % (unsigned)n_tiles);
      t /= (unsigned)n_tiles;
      g = (int)(t % (unsigned)Hkv);
      b = (int)(t / (unsigned)Hkv);
    } else if (((unsigned)B * (unsigned)Hkv) % kXcds == 0) {
      // Tile-major, heavier tiles first; for tile rank t, XCD x takes the KV
      // groups bg with (bg + t / kRotRun) % 8 == x (all G query heads of each):
      // a group stays on one XCD for kRotRun consecutive tiles (which select
      // mostly the same blocks, so they share its L2) and then moves on, so
      // every group's work is spread over all XCDs.
      if (blockIdx.x >= total) return;
      const unsigned x = blockIdx.x % kXcds, idx = blockIdx.x / kXcds;
      const unsigned per_tile = ((unsigned)B * (unsigned)Hq) / kXcds;
      const unsigned tr = idx / per_tile, rem = idx % per_tile;
      tile = n_tiles - 1 - (int)tr;
      hh = (int)(rem % G);
      const unsigned rot = (tr / kRotRun) % kXcds;
      const unsigned bg = (x + kXcds - rot) % kXcds + kXcds * (rem / G);
      b = (int)(bg / (unsigned)Hkv);
      g = (int)(bg % (unsigned)Hkv);
    } else {
      // Tile-major with the (batch, head) index rotated by one per tile.
      if (blockIdx.x >= total) return;
      const unsigned R = (unsigned)B * (unsigned)Hq;
      const unsigned tr = blockIdx.x / R;
      const unsigned r = (blockIdx.x % R + tr) % R;
      tile = n_tiles - 1 - (int)tr;
      b = (int)(r / (unsigned)Hq);
      hh = (int)(r % (unsigned)Hq) % (int)G;
      g = (int)(r % (unsigned)Hq) / (int)G;
    }
    const int h = g * (int)G + hh;

    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63;
    const int jq = lane & 31, hf = lane >> 5;
    const int q0 = tile * kTileQ;
    const int q_last = min(q0 + kTileQ - 1, N - 1);
    const int qw0 = q0 + wave * 32;          // first query row of this wave
    const int qrow = qw0 + jq;               // this lane's query row

    const uint16_t* kh = k + (size_t)(b * Hkv + g) * N * kHeadDim;
    const uint16_t* vh = v + (size_t)(b * Hkv + g) * N * kHeadDim;

    // Q^T fragments (B operand of S^T = K Q^T), kept in registers.
    bf16x8 qf[8];
    {
      const uint16_t* qp = q + ((size_t)(b * Hq + h) * N + qrow) * kHeadDim + 8 * hf;
  #pragma unroll
      for (int s = 0; s < 8; ++s)
        qf[s] = as_bf16x8(qrow < N ? *(const uint4*)(qp + 16 * s) : make_uint4(0, 0, 0, 0));
    }

    // The sub-blocks to visit.
    const int32_t* lst = nullptr;
    int n_steps;
    if (MODE == kSparse) {
      const int seg = q0 / Ls;
      lst = bidx + ((size_t)(b * Hq + h) * CS + seg) * kmax;
      const int c = min(max(bcnt[(size_t)(b * Hq + h) * CS + seg], 0), kmax);
      n_steps = valid_prefix<SUB>(lst, c, CB, q_last, lane) * SUB;
    } else if (MODE == kDenseCausal) {
      n_steps = q_last / kSub + 1;
    } else {
      n_steps = (N + kSub - 1) / kSub;
    }
    auto step_key0 = [&](int i) -> int {
      if (MODE == kSparse) return (SUB == 1 ? lst[i] : lst[i >> 1] * SUB + (i & 1)) * kSub;
      return i * kSub;
    };

    // byte offsets of this lane's stage copies inside a 64-row block
    uint32_t koff[4], voff;
    stage_offsets<4>(wave, lane, koff, voff);

    f32x16 oacc[4];
  #pragma unroll
    for (int d = 0; d < 4; ++d)
  #pragma unroll
      for (int r = 0; r < 16; ++r) oacc[d][r] = 0.0f;
    float m_i = -INFINITY, l_i = 0.0f;

    // Two-stage LDS ring filled directly from global memory.  Step i waits for
    // its stage (the 8 loads of step i+1 may still be in flight), computes, and
    // after a second barrier refills the stage with step i+2.  Even steps use
    // stage0, odd steps stage1.
    auto step = [&](const int i, unsigned char* st) {
      if (i + 1 < n_steps) EI_WAIT_VMCNT(8); else EI_WAIT_VMCNT(0);
      __syncthreads();
      const int k0 = step_key0(i);
      const bool active = (MODE == kDenseFull) || (k0 <= qw0 + 31);
      if (active && qw0 < N)
        compute_step<MODE>(st, k0, qw0, qrow, N, jq, hf, lane, qf, sc_log2, oacc, m_i, l_i);
      if (i + 2 < n_steps) {
        __syncthreads();   // every wave is done reading this stage
        issue_stage<4>(st, kh, vh, step_key0(i + 2), N, wave, lane, koff, voff);
      }
    };
    // Q fragments (and the list) have landed before any stage copy is issued,
    // so no later wait on them covers the copies in flight.
    EI_WAIT_VMCNT(0);
    if (n_steps > 0) issue_stage<4>(stage0, kh, vh, step_key0(0), N, wave, lane, koff, voff);
    if (n_steps > 1) issue_stage<4>(stage1, kh, vh, step_key0(1), N, wave, lane, koff, voff);
    if (pers && kmax * SUB <= kShortItem) {   // the next item's ticket (own queue)
      if (threadIdx.x == 0) ticket = atomicAdd(&sched[x0], 1u);
      taken = true;
    }
    for (int i = 0; i < n_steps; i += 2) {
      step(i, stage0);
      if (i + 1 < n_steps) step(i + 1, stage1);
    }

    if (qrow < N) store_rows(o, (size_t)(b * Hq + h) * N + qrow, hf, oacc, l_i);
    if (!pers) return;
    __syncthreads();   // every wave is done with the stages (and the item)
  }
}

// ---------------------------------------------------------------------------
// Small launches.  A launch of few tiles leaves most CUs idle while each of
// its waves walks its tile's keys in turn (a 1024-token, 4-head layer: 32
// workgroups of up to 16 steps of ~1 us).  Here a workgroup takes a 32-row tile
// and its four waves every fourth step of the tile's keys, each with a stage
// of its own in LDS (no barrier inside the loop: a wave waits for its own
// copies only, the next step's K copied once this step's scores have been
// read, its V after the last product); the four partial (m, l, O) are merged
// through LDS at the end.  The same rows, blocks and arithmetic per step as
// attn_kernel; the result differs by the order of the sums and by the rounding
// of the probabilities to bf16, against the wave's own running maximum.
constexpr int kSplitWaves = kThreads / kWave;
constexpr int kSplitTileQ = 32;

// The wave's own 64-row K (or V) tile: four groups of four 1 KB copies.
__device__ __forceinline__ void issue_tile(unsigned char* dst, const uint16_t* __restrict__ src,
                                           int k0, int N, int lane, const uint32_t* off,
                                           bool is_v) {
  const int kc = min(k0, N - 1);   // (as in issue_stage)
  const unsigned char* sb = (const unsigned char*)src + (size_t)kc * kRowBytes;
  const uint32_t d0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)dst);
  if (k0 + kSub <= N) {
#pragma unroll
    for (int g = 0; g < 4; ++g) copy_rows_to_lds<4>(sb + 4096 * g, off, d0 + 4096 * g);
    return;
  }
  // (opaque: the 16 row offsets are formed here, not kept across the loop)
  asm volatile("" : "+v"(lane));
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const int row = 4 * j + (lane >> 4), pos = lane & 15;
    copy_row_to_lds(sb, (uint32_t)((min(k0 + row, N - 1) - kc) * kRowBytes) +
                            16 * (is_v ? swz_v(row, pos) : swz(row, pos)),
                    d0 + 1024 * j);
  }
}

template <int MODE, int SUB>
__global__ __launch_bounds__(kThreads, 1) void attn_split_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
    const uint16_t* __restrict__ v, uint16_t* __restrict__ o, int Hq, int Hkv, int N, int n_tiles,
    int Ls, int CS, int CB, float sc_log2, const int32_t* __restrict__ bidx,
    const int32_t* __restrict__ bcnt, int kmax) {
  __shared__ __attribute__((aligned(1024))) unsigned char stages[kSplitWaves][kStageBytes];
  __shared__ float part_m[kSplitWaves][kSplitTileQ], part_l[kSplitWaves][kSplitTileQ];
  const int rows = gridDim.x / n_tiles;   // (batch, query head) pairs
  const int tile = n_tiles - 1 - (int)blockIdx.x / rows, bh = (int)blockIdx.x % rows;
  const int b = bh / Hq, h = bh % Hq, g = h / (Hq / Hkv);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int jq = lane & 31, hf = lane >> 5;
  const int q0 = tile * kSplitTileQ, q_last = min(q0 + kSplitTileQ - 1, N - 1), qrow = q0 + jq;
  const uint16_t* kh = k + (size_t)(b * Hkv + g) * N * kHeadDim;
  const uint16_t* vh = v + (size_t)(b * Hkv + g) * N * kHeadDim;

  bf16x8 qf[8];
  {
    const uint16_t* qp = q + ((size_t)bh * N + qrow) * kHeadDim + 8 * hf;
#pragma unroll
    for (int s = 0; s < 8; ++s)
      qf[s] = as_bf16x8(qrow < N ? *(const uint4*)(qp + 16 * s) : make_uint4(0, 0, 0, 0));
  }
  const int32_t* lst = nullptr;
  int n_steps;
  if (MODE == kSparse) {
    const int64_t row = (int64_t)bh * CS + q0 / Ls;
    lst = bidx + row * kmax;
    n_steps = valid_prefix<SUB>(lst, min(max(bcnt[row], 0), kmax), CB, q_last, lane) * SUB;
  } else {
    n_steps = MODE == kDenseCausal ? q_last / kSub + 1 : (N + kSub - 1) / kSub;
  }
  // lane t: the list entry of the wave's t-th step (read here once: a load in
  // the loop would be waited for behind the copies)
  int lv = 0;
  if (MODE == kSparse) {
    const int e = (wave + kSplitWaves * lane) / SUB;
    if (e < n_steps / SUB) lv = lst[e];
    asm volatile("" : "+v"(lv));
  }
  auto step_key0 = [&](int i) -> int {
    if (MODE != kSparse) return i * kSub;
    const int blk = __builtin_amdgcn_readlane(lv, (i / kSplitWaves) & (kWave - 1));
    return (SUB == 1 ? blk : blk * SUB + (i & 1)) * kSub;
  };
  unsigned char* st = stages[wave];
  uint32_t koff[4], voff[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    koff[j] = (uint32_t)((lane >> 4) * kRowBytes + 16 * swz(4 * j + (lane >> 4), lane & 15));
    voff[j] = (uint32_t)((lane >> 4) * kRowBytes + 16 * swz_v(lane >> 4, lane & 15));
  }

  f32x16 oacc[4];
#pragma unroll
  for (int d = 0; d < 4; ++d)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[d][r] = 0.0f;
  float m_i = -INFINITY, l_i = 0.0f;

  EI_WAIT_VMCNT(0);   // the Q operands: no later wait covers copies in flight
  int k0 = 0;
  if (wave < n_steps) {
    k0 = step_key0(wave);
    issue_tile(st, kh, k0, N, lane, koff, false);
    issue_tile(st + kTileBytes, vh, k0, N, lane, voff, true);
  }
  for (int i = wave; i < n_steps; i += kSplitWaves) {
    const bool more = i + kSplitWaves < n_steps;
    const int kn = more ? step_key0(i + kSplitWaves) : 0;
    EI_WAIT_VMCNT(16);   // K has landed (V's 16 copies may be in flight)
    asm volatile("" ::: "memory");
    // (every LDS read of a tile has returned before its copies are issued)
    auto next_k = [&]() {
      EI_WAIT_LGKM0();
      if (more) issue_tile(st, kh, kn, N, lane, koff, false);
    };
    auto wait_v = [&]() {
      if (more) EI_WAIT_VMCNT(16); else EI_WAIT_VMCNT(0);
      asm volatile("" ::: "memory");
    };
    if (MODE == kDenseFull || k0 <= q_last) {
      compute_step<MODE, true>(st, k0, q0, qrow, N, jq, hf, lane, qf, sc_log2, oacc, m_i, l_i,
                               next_k, wait_v);
    } else {
      next_k();
      wait_v();
    }
    EI_WAIT_LGKM0();
    if (more) issue_tile(st + kTileBytes, vh, kn, N, lane, voff, true);
    k0 = kn;
  }

  // Merge: each wave leaves its O in its own stage (every read and copy of
  // which is done), then takes 32 of the 128 dims of all four.
  const float l = l_i + __shfl_xor(l_i, 32);
  if (hf == 0) {
    part_m[wave][jq] = m_i;
    part_l[wave][jq] = l;
  }
#pragma unroll
  for (int d = 0; d < 4; ++d)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      *(float4*)(st + ((d * 4 + r) * kWave + lane) * 16) =
          make_float4(oacc[d][4 * r], oacc[d][4 * r + 1], oacc[d][4 * r + 2], oacc[d][4 * r + 3]);
  __syncthreads();
  float m = part_m[0][jq];
#pragma unroll
  for (int w = 1; w < kSplitWaves; ++w) m = fmaxf(m, part_m[w][jq]);
  float f[kSplitWaves], lsum = 0.0f;
#pragma unroll
  for (int w = 0; w < kSplitWaves; ++w) {
    const float mw = part_m[w][jq];
    f[w] = mw == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(mw - m);
    lsum += f[w] * part_l[w][jq];
  }
  const float inv = lsum > 0.0f ? 1.0f / lsum : 0.0f;
  if (qrow >= N) return;
  uint16_t* op = o + ((size_t)bh * N + qrow) * kHeadDim + 32 * wave + 4 * hf;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    float4 a = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll
    for (int w = 0; w < kSplitWaves; ++w) {
      const float4 x = *(const float4*)(stages[w] + ((wave * 4 + r) * kWave + lane) * 16);
      a.x += f[w] * x.x;
      a.y += f[w] * x.y;
      a.z += f[w] * x.z;
      a.w += f[w] * x.w;
    }
    *(uint2*)(op + 8 * r) =
        make_uint2(pack_bf16x2(a.x * inv, a.y * inv), pack_bf16x2(a.z * inv, a.w * inv));
  }
}

// Which launches take the split.  Its 32-row tiles run one to a CU (128 KB of
// LDS) and each copies its keys for itself, so the choice lies with the rounds
// they make on the CUs and the steps a tile has (us, 128-row / split tiles):
//  - up to 128 tokens, over all keys 96: little to share out (64 tokens 5.0 /
//    6.1; 8 heads, 120 causal 6.7 / 6.7, 80 over all keys 6.5 / 6.6).  Lists
//    would gain from 97 (7.3 / 7.1), but a sparse launch follows the causal one
//    wherever its lists can hold every block: the two are then bitwise equal;
//  - one round: from there always (16 heads, 129 causal 7.0 / 6.5, 512 14.6 /
//    9.0; 4 heads, 2048 42.9 / 18.9; over lists of six steps 12.9 / 9.3; 8
//    heads, 97 tokens, all keys 7.2 / 6.6);
//  - two rounds (at most kSplitMaxTiles 128-row tiles, half the CUs): the
//    second has to be paid for by the steps that a wave does not make.  Causal
//    tiles pay from 9 (7: 32 heads, 400 tokens 12.3 / 13.7; 8: 28 heads, 512
//    15.0 / 14.2, 481 14.3 / 14.1; 9: 16 heads, 517 14.6 / 11.6; 64: 4 heads,
//    4096 82 / 40), tiles over all keys, equally long, from 14 (9: 16 heads, 517
//    16.5 / 17.9; 13: 769 21.4 / 21.2; 15: 900 23.9 / 21.7; 64: 4 heads, 4096
//    81 / 55).  Lists of capacity C steps hold C / 3 and more at the default
//    cap; those far shorter than the sequence are as equal as full tiles, with
//    few steps (C = 14: 8 heads, 1531 tokens 23.3 / 19.4, 2048 21.1 / 21.5, 1
//    head, 16384 14.0 / 18.2; C = 26: 2 heads, 5000 37.8 / 27.7, 1 head, 16384
//    19.3 / 22.5; C = 98: 1 head, 16384 49.5 / 43.3).  How long the lists are the
//    host does not know.  Of 3368 sparse launches of two rounds that the rule
//    gives to the split, 116 lost by it, 29 of them by more than an eighth and
//    the worst 13.1 / 16.8 (8 heads, 1673, C = 14); in all of these the lists
//    held their least, C / 3 or so, of up to 18 steps.  With lists 5% longer
//    on average none of 485 lost, and the median gained 1.58x.
constexpr int kSplitMaxTiles = 128, kSplitRound = 2 * kSplitMaxTiles;
static_assert(kSplitMaxTiles * kTileQ / kSub <= kSplitWaves * kWave, "a lane per step of a wave");
template <int MODE, int SUB>
bool split_tiles(const AttnShape& s) {
  const int64_t rows = (int64_t)s.B * s.Hq, steps = (s.N + kSub - 1) / kSub;
  if (rows * ((s.N + kTileQ - 1) / kTileQ) > kSplitMaxTiles ||
      s.N <= (MODE == kDenseFull ? 96 : 128))
    return false;
  if (rows * ((s.N + kSplitTileQ - 1) / kSplitTileQ) <= kSplitRound) return true;
  if (steps < (MODE == kDenseFull ? 14 : 9)) return false;
  const int64_t cap = (int64_t)s.kmax * SUB;
  return MODE != kSparse || (cap >= 9 && steps <= (cap < 24 ? 2 : 4) * cap);
}

template <int MODE, int SUB>
hipError_t launch_split_t(const uint16_t* q, const uint16_t* k, const uint16_t* v,
                          const AttnShape& s, const int32_t* bidx, const int32_t* bcnt,
                          uint16_t* o, hipStream_t stream) {
  const int n_tiles = (s.N + kSplitTileQ - 1) / kSplitTileQ;
  const float sc_log2 = (float)((double)s.softmax_scale * 1.4426950408889634);
  hipLaunchKernelGGL((attn_split_kernel<MODE, SUB>), dim3((unsigned)(s.B * s.Hq * n_tiles)),
                     dim3(kThreads), 0, stream, q, k, v, o, s.Hq, s.Hkv, s.N, n_tiles, s.Ls, s.CS,
                     s.CB, sc_log2, bidx, bcnt, s.kmax);
  return hipGetLastError();
}

// The persistent plan for a shape, if its KV groups tile the XCDs.
bool make_plan(const AttnShape& s, int n_tiles, XcdPlan& pl) {
  const unsigned NG = (unsigned)(s.B * s.Hkv), G = (unsigned)(s.Hq / s.Hkv);
  if (NG % kXcds == 0) {
    pl.S = 1;
    pl.ngx = NG / kXcds;
    for (unsigned x = 0; x < kXcds; ++x) pl.per_x[x] = (unsigned)n_tiles * G * pl.ngx;
    return true;
  }
  if (kXcds % NG != 0) return false;
  pl.S = kXcds / NG;
  pl.ngx = 1;
  const unsigned cyc = pl.S * kRun, full = (unsigned)n_tiles / cyc, rem = (unsigned)n_tiles % cyc;
  for (unsigned x = 0; x < kXcds; ++x) {
    const unsigned part = x / NG;
    const unsigned tail = rem > part * kRun ? min(rem - part * kRun, kRun) : 0u;
    pl.per_x[x] = G * (full * kRun + tail);
  }
  return true;
}

// Workgroups of the persistent grid: two per CU of the current device.
int persistent_grid() {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      cus <= 0)
    return 0;
  return 2 * cus;
}

template <int MODE, int SUB>
hipError_t launch_t(const uint16_t* q, const uint16_t* k, const uint16_t* v, const AttnShape& s,
                    const int32_t* bidx, const int32_t* bcnt, uint16_t* o, uint32_t* sched,
                    bool sched_zeroed, hipStream_t stream) {
  if (split_tiles<MODE, SUB>(s)) return launch_split_t<MODE, SUB>(q, k, v, s, bidx, bcnt, o, stream);
  const int n_tiles = (s.N + kTileQ - 1) / kTileQ;
  const int64_t total = (int64_t)s.B * s.Hq * n_tiles;
  int64_t grid = (total + kXcds - 1) / kXcds * kXcds;
  XcdPlan plan{};
  int pgrid = 0;
  // A launch whose items all fit the persistent grid at once has nothing to
  // queue or steal: the static grid then saves the items' atomics and the
  // counters' reset (a launch of its own, 4 us, outside the one-call path).
  if (MODE == kSparse && sched != nullptr && make_plan(s, n_tiles, plan) &&
      (pgrid = persistent_grid()) > 0 && total > pgrid) {
    if (!sched_zeroed)
      hipLaunchKernelGGL(sched_reset_kernel, dim3(1), dim3(kWave), 0, stream, sched);
    grid = (int64_t)pgrid;
  } else {
    sched = nullptr;
  }
  if (!launch_fits(grid, kThreads)) return hipErrorInvalidConfiguration;
  const float sc_log2 = (float)((double)s.softmax_scale * 1.4426950408889634);
  hipLaunchKernelGGL((attn_kernel<MODE, SUB>), dim3((unsigned)grid), dim3(kThreads), 0, stream,
                     q, k, v, o, s.B, s.Hq, s.Hkv, s.N, n_tiles, s.Ls, s.CS, s.CB, sc_log2, bidx,
                     bcnt, s.kmax, sched, plan);
  return hipGetLastError();
}


// ---------------------------------------------------------------------------
// GQA-union tiles.  One workgroup of 8 waves takes the same 128-row query tile
// of two query heads that share a KV head (waves 0-3 the first, 4-7 the
// second).  The heads' block lists are merged into their union (a bitmap over
// the key blocks, compacted in ascending order); each union block is copied
// into LDS once, and the waves of a head that did not select it skip its
// compute while still taking part in the barriers.  Every head visits its own
// blocks in ascending order with compute_step, so the output equals
// attn_kernel's bit for bit.
constexpr int kUnionThreads = 2 * kThreads;
constexpr int kUnionWords = kUnionMaxBlocks / 32;

template <int SUB>
__global__ __launch_bounds__(kUnionThreads, 1) void attn_union_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
    const uint16_t* __restrict__ v, uint16_t* __restrict__ o, int B, int Hq, int Hkv, int N,
    int n_tiles, int Ls, int CS, int CB, float sc_log2, const int32_t* __restrict__ bidx,
    const int32_t* __restrict__ bcnt, int kmax) {
  __shared__ __attribute__((aligned(1024))) unsigned char stage0[kStageBytes];
  __shared__ __attribute__((aligned(1024))) unsigned char stage1[kStageBytes];
  __shared__ uint32_t sel_bits[2][kUnionWords];     // the two heads' selected blocks
  __shared__ uint32_t word_off[kUnionWords + 1];    // union entries before each word
  __shared__ uint32_t ulist[2 * kUnionMaxList];     // block | head-0 bit 30 | head-1 bit 31

  // Tile-major, heavier tiles first, the (batch, KV head, pair) index rotated
  // by one per tile.
  const int G = Hq / Hkv, npair = (G + 1) / 2;
  const unsigned R = (unsigned)B * (unsigned)Hkv * (unsigned)npair;
  if (blockIdx.x >= R * (unsigned)n_tiles) return;
  const unsigned tr = blockIdx.x / R;
  const unsigned rr = (blockIdx.x % R + tr) % R;
  const int tile = n_tiles - 1 - (int)tr;
  const int pair = (int)(rr % (unsigned)npair);
  const int bg = (int)(rr / (unsigned)npair);
  const int b = bg / Hkv, g = bg % Hkv;

  const int tid = threadIdx.x;
  const int wave = tid >> 6, lane = tid & 63;
  const int side = wave >> 2, wq = wave & 3;
  const int jq = lane & 31, hf = lane >> 5;
  const bool has_head = 2 * pair + side < G;        // the second side of an odd G is empty
  const int h = g * G + min(2 * pair + side, G - 1);
  const int q0 = tile * kTileQ;
  const int q_last = min(q0 + kTileQ - 1, N - 1);
  const int qw0 = q0 + wq * 32;
  const int qrow = qw0 + jq;

  const uint16_t* kh = k + (size_t)(b * Hkv + g) * N * kHeadDim;
  const uint16_t* vh = v + (size_t)(b * Hkv + g) * N * kHeadDim;

  bf16x8 qf[8];
  {
    const uint16_t* qp = q + ((size_t)(b * Hq + h) * N + qrow) * kHeadDim + 8 * hf;
#pragma unroll
    for (int s = 0; s < 8; ++s)
      qf[s] = as_bf16x8(qrow < N ? *(const uint4*)(qp + 16 * s) : make_uint4(0, 0, 0, 0));
  }

  // The union of the two heads' valid list prefixes, ascending.
  const int seg = q0 / Ls;
  for (int i = tid; i < 2 * kUnionWords; i += kUnionThreads) (&sel_bits[0][0])[i] = 0u;
  __syncthreads();
  for (int sd = 0; sd < 2; ++sd) {
    if (2 * pair + sd >= G) continue;
    const int hs = g * G + 2 * pair + sd;
    const int32_t* lst = bidx + ((size_t)(b * Hq + hs) * CS + seg) * kmax;
    const int c = min(max(bcnt[(size_t)(b * Hq + hs) * CS + seg], 0), kmax);
    const int nv = valid_prefix<SUB>(lst, c, CB, q_last, lane);
    for (int e = tid; e < nv; e += kUnionThreads) {
      const int blk = lst[e];
      atomicOr(&sel_bits[sd][blk >> 5], 1u << (blk & 31));
    }
  }
  __syncthreads();
  const int nw = (CB + 31) / 32;
  if (wave == 0) {
    uint32_t cnt[4], S = 0;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int wd = 4 * lane + t;
      cnt[t] = wd < nw ? (uint32_t)__popc(sel_bits[0][wd] | sel_bits[1][wd]) : 0u;
      S += cnt[t];
    }
    const uint32_t pre = wave_incl_scan_u32(S);
    uint32_t off = pre - S;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      word_off[4 * lane + t] = off;
      off += cnt[t];
    }
    if (lane == kWave - 1) word_off[kUnionWords] = pre;
  }
  __syncthreads();
  for (int wd = tid; wd < nw; wd += kUnionThreads) {
    const uint32_t a = sel_bits[0][wd], c2 = sel_bits[1][wd];
    uint32_t u = a | c2, p = word_off[wd];
    while (u != 0u) {
      const int bit = __builtin_ctz(u);
      u &= u - 1u;
      ulist[p++] = (uint32_t)(32 * wd + bit) | (((a >> bit) & 1u) << 30) |
                   (((c2 >> bit) & 1u) << 31);
    }
  }
  __syncthreads();
  const int n_steps = (int)word_off[kUnionWords] * SUB;
  auto entry = [&](int i) -> uint32_t { return ulist[SUB == 1 ? i : i >> 1]; };
  auto key0 = [&](uint32_t e, int i) -> int {
    const int blk = (int)(e & 0x3fffffffu);
    return (SUB == 1 ? blk : blk * SUB + (i & 1)) * kSub;
  };

  uint32_t koff[2], voff;
  stage_offsets<2>(wave, lane, koff, voff);

  f32x16 oacc[4];
#pragma unroll
  for (int d = 0; d < 4; ++d)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[d][r] = 0.0f;
  float m_i = -INFINITY, l_i = 0.0f;

  // The ring of attn_kernel with four copies per wave and stage.
  auto step = [&](const int i, unsigned char* st) {
    if (i + 1 < n_steps) EI_WAIT_VMCNT(4); else EI_WAIT_VMCNT(0);
    __syncthreads();
    const uint32_t e = entry(i);
    const int k0 = key0(e, i);
    const bool mine = has_head && ((e >> (30 + side)) & 1u) != 0u;
    if (mine && k0 <= qw0 + 31 && qw0 < N)
      compute_step<kSparse>(st, k0, qw0, qrow, N, jq, hf, lane, qf, sc_log2, oacc, m_i, l_i);
    if (i + 2 < n_steps) {
      __syncthreads();   // every wave is done reading this stage
      issue_stage<2>(st, kh, vh, key0(entry(i + 2), i + 2), N, wave, lane, koff, voff);
    }
  };
  EI_WAIT_VMCNT(0);
  if (n_steps > 0) issue_stage<2>(stage0, kh, vh, key0(entry(0), 0), N, wave, lane, koff, voff);
  if (n_steps > 1) issue_stage<2>(stage1, kh, vh, key0(entry(1), 1), N, wave, lane, koff, voff);
  for (int i = 0; i < n_steps; i += 2) {
    step(i, stage0);
    if (i + 1 < n_steps) step(i + 1, stage1);
  }

  if (!has_head || qrow >= N) return;
  store_rows(o, (size_t)(b * Hq + h) * N + qrow, hf, oacc, l_i);
}

template <int SUB>
hipError_t launch_union_t(const uint16_t* q, const uint16_t* k, const uint16_t* v,
                          const AttnShape& s, const int32_t* bidx, const int32_t* bcnt,
                          uint16_t* o, hipStream_t stream) {
  // (bitwise the per-head kernel's output, so also the same kernel here)
  if (split_tiles<kSparse, SUB>(s)) return launch_split_t<kSparse, SUB>(q, k, v, s, bidx, bcnt, o, stream);
  const int n_tiles = (s.N + kTileQ - 1) / kTileQ;
  const int npair = (s.Hq / s.Hkv + 1) / 2;
  const int64_t grid = (int64_t)s.B * s.Hkv * npair * n_tiles;
  if (!launch_fits(grid, kUnionThreads)) return hipErrorInvalidConfiguration;
  const float sc_log2 = (float)((double)s.softmax_scale * 1.4426950408889634);
  hipLaunchKernelGGL((attn_union_kernel<SUB>), dim3((unsigned)grid), dim3(kUnionThreads), 0,
                     stream, q, k, v, o, s.B, s.Hq, s.Hkv, s.N, n_tiles, s.Ls, s.CS, s.CB,
                     sc_log2, bidx, bcnt, s.kmax);
  return hipGetLastError();
}

}  // namespace

bool attention_union_supported(const AttnShape& s) {
  return s.kmax <= kUnionMaxList && s.CB <= kUnionMaxBlocks;
}

hipError_t launch_attention_union(const uint16_t* q, const uint16_t* k, const uint16_t* v,
                                  const AttnShape& s, const int32_t* block_idx,
                                  const int32_t* block_cnt, uint16_t* o, hipStream_t stream) {
  if (!attention_union_supported(s)) return hipErrorInvalidValue;
  return s.Lb == 2 * kSub ? launch_union_t<2>(q, k, v, s, block_idx, block_cnt, o, stream)
                          : launch_union_t<1>(q, k, v, s, block_idx, block_cnt, o, stream);
}

hipError_t launch_attention(const uint16_t* q, const uint16_t* k, const uint16_t* v,
                            const AttnShape& s, AttnMode mode, const int32_t* block_idx,
                            const int32_t* block_cnt, uint16_t* o, void* sched_ws,
                            bool sched_zeroed, hipStream_t stream) {
  if (s.B * (int64_t)s.Hq * ((s.N + kTileQ - 1) / kTileQ) >= (int64_t)1 << 31)
    return hipErrorInvalidValue;
  uint32_t* sched = (uint32_t*)sched_ws;
  switch (mode) {
    case kSparse:
      return s.Lb == 2 * kSub
                 ? launch_t<kSparse, 2>(q, k, v, s, block_idx, block_cnt, o, sched, sched_zeroed, stream)
                 : launch_t<kSparse, 1>(q, k, v, s, block_idx, block_cnt, o, sched, sched_zeroed,
                                        stream);
    case kDenseCausal:
      return launch_t<kDenseCausal, 1>(q, k, v, s, nullptr, nullptr, o, nullptr, false, stream);
    default:
      return launch_t<kDenseFull, 1>(q, k, v, s, nullptr, nullptr, o, nullptr, false, stream);
  }
}

}  // namespace ei
