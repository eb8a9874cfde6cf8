// Tree-masked attention for one Progressive Tree Drafting step on gfx950.
//
// Sec. 3.1 "Tree Construction" + Sec. 3.2: every packed tree node attends to
// the committed prefix and to its own ancestors (pi(v) = {v} u pi(P(v))) only.
// For sequence b, KV head g and query row r = i*G + hg (node i, query head
// h = g*G + hg), the keys are cache rows [0, kv_len) plus kv_len + a for every
// ancestor-or-self a of node i; node i's own K/V row is kv_len + i.
//
// Kernels
//   k_attn_mfma    bf16 q/k/v.  One workgroup = (b, g, row pass, KV split);
//                  8 waves (2 per SIMD), each owning up to 32 query rows.  K/V
//                  stream HBM -> LDS with asynchronous copies into a ring of
//                  ten 32-key sub-tiles (all 160 KB of LDS), shared by every
//                  query row of the GQA group; V is read transposed straight
//                  from its natural layout with ds_read_b64_tr_b16.  Scores
//                  are computed transposed, S^T = K Q^T, and the output as
//                  O^T = V^T P^T, so each lane owns one query column in both
//                  accumulators and the online-softmax rescale is lane-local;
//                  the softmax row sums are one more MFMA of P with an
//                  all-ones operand.  MFMA: v_mfma_f32_16x16x32_bf16, fp32
//                  accumulation.
//                  Trees of up to 128 nodes need no mask pass: each lane
//                  holds two parent[] entries and walks its rows' ancestor
//                  chains with wave shuffles.  With the keys split over
//                  several workgroups, each writes fp32 partials (m, l, O).
//   k_attn_combine merges split-KV partials in a fixed split order.
//   k_attn_f32     fp32 inputs: v_mfma_f32_16x16x4_f32, fp32 throughout.
#include <math.h>

#include <algorithm>
#include <mutex>
#include <type_traits>

#include "ptd_async.hpp"
#include "ptd_common.hpp"
#include "ptd_internal.hpp"

namespace {

using ptd::dma16;
using ptd::dma16_s;
using ptd::lds_addr;
using ptd::lds_barrier;
using ptd::wait_vmcnt;
using ptd::wait_vmcnt_le;

using bf16x8 = __bf16 __attribute__((ext_vector_type(8)));
using f32x4 = float __attribute__((ext_vector_type(4)));
using u32x4 = uint32_t __attribute__((ext_vector_type(4)));
using u32x2 = uint32_t __attribute__((ext_vector_type(2)));

constexpr int kThreads = 512;   // 8 waves: two per SIMD
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kNegBig = -1.0e30f;  // running-max start: finite, below any score
// A query block of a tile in which some softmax weight p exceeds this
// fraction of its query row's sum so far carries p into the PV product as
// bf16 hi + lo rather than bf16 (see k_attn_mfma).
constexpr float kPreciseFrac = 1.0f / 16.0f;

struct AttnParams {
  const void* q;
  const void* k;
  const void* v;
  const int32_t* kv_len;
  const int32_t* parent;  // [B][T]
  const int32_t* tree_len;  // [B] or null: nodes at index >= tree_len[b] are padding
  const float* k_scale;     // [Hkv] or null (8-bit caches): key = code value * k_scale[g]
  const float* v_scale;     // [Hkv] or null: value = code value * v_scale[g]
  const uint64_t* mask;   // [B][T][W] ancestor words (trees of more than 128 nodes; fp32 when given)
  void* out;
  float* part_o;    // [S][B][Hkv][M][D]
  float2* part_ml;  // [S][B][Hkv][M]: (running max * c, sum of p)
  int32_t* dev_status;
  int B, T, Hq, Hkv, G, M, L_cap, W;
  int splits, passes, rows_per_pass;
  // paged caches: k and v are [num_pages][Hkv][2^page_shift][D] and row r of
  // sequence b lives in page page_table[b][r >> page_shift]; null: contiguous
  const int32_t* page_table;
  int page_shift, max_pages, num_pages;
  float scale;  // softmax scale
  float c;      // scale * log2(e)
  float precise;  // kPreciseFrac, or a smaller share
  int out_bf16;
};

// Keys of a sequence are [0, N), N = kv_len + T, cut into `splits` chunks of
// this size (a multiple of 32, the key granularity of one MFMA step).
__host__ __device__ inline int chunk_size(int N, int splits) {
  const int c = (N + splits - 1) / splits;
  return (c + 31) & ~31;
}

// Live nodes of sequence b (the rest of the T slots are padding).
__device__ inline int live_nodes(const AttnParams& p, int b) {
  return p.tree_len ? min(max(p.tree_len[b], 0), p.T) : p.T;
}

__device__ inline void logical_block(int bid, int nblocks, int npairs, bool by_size, int& id) {
  // Workgroups are dealt round-robin over the 8 XCDs (block i to XCD i mod 8)
  // and each XCD runs its share in block order.  The items of one (b, g) pair
  // (its row passes and KV splits) share keys and query rows, so they stay on
  // one XCD (one L2), consecutive.  With the sequences ordered by size
  // (by_size), the pairs are dealt round-robin over the XCDs too (pair q to
  // XCD q mod 8), so every XCD gets a like share of long and short sequences
  // and runs its own largest first; otherwise each XCD takes a contiguous
  // range of pairs.
  if (by_size && (npairs & 7) == 0 && (nblocks & 7) == 0) {
    const int ips = nblocks / npairs;  // items per pair
    const int x = bid & 7, j = bid >> 3;
    id = (x + 8 * (j / ips)) * ips + j % ips;
  } else if ((nblocks & 7) == 0) {
    id = (bid & 7) * (nblocks >> 3) + (bid >> 3);
  } else {
    id = bid;
  }
}

// ===========================================================================
// MFMA path
// ===========================================================================
// Max / sum of a lane's value and that of lane ^ 32 (or ^ 16), on the VALU
// (gfx950 v_permlane32_swap / v_permlane16_swap: with both operands holding
// the value, the two results are the value of the lane and of its partner).
__device__ __forceinline__ float max_xor32(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float max_xor16(float v) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum_xor32(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float sum_xor16(float v) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

using i16x4 = short __attribute__((ext_vector_type(4)));

__device__ __forceinline__ i16x4 lds_read_tr16(const unsigned char* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((PTD_LDS i16x4*)p);
}

using i32x2 = int __attribute__((ext_vector_type(2)));
// Transpose read of bytes (ds_read_b64_tr_b8): in each 16-lane group, lane i
// receives byte i mod 8 of the 8 bytes read by the group's lanes 2j + i / 8,
// j = 0..7, as its bytes j.
__device__ __forceinline__ u32x2 lds_read_tr8(const unsigned char* p) {
  return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr8_b64_v2i32((PTD_LDS i32x2*)p));
}
// Eight OCP E4M3 values (bytes 0..7 of w) as eight bf16, exactly (every E4M3
// value is a bf16 value): gfx950 v_cvt_scalef32_pk_bf16_fp8 with scale 1.
__device__ __forceinline__ bf16x8 e4m3x8_to_bf16(u32x2 w) {
  const u32x4 r = {
      __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w[0], 1.0f, false)),
      __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w[0], 1.0f, true)),
      __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w[1], 1.0f, false)),
      __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w[1], 1.0f, true))};
  return __builtin_bit_cast(bf16x8, r);
}

// LDS layout of one 32-key sub-tile: K rows then V rows, each [32][D] of
// ES-byte elements (bf16, or E4M3 for 8-bit caches), row-major with the
// 16-byte chunks of row r stored XOR-permuted (CH = D*ES/16 chunks per row).
// bf16, D = 128 (16 chunks): K rows by r mod 16, V rows by f(r) = ((r mod 8)
// << 1) | bit 3 of r.  The K-operand reads (ds_read_b128: 16 rows x one
// chunk per 16 lanes) are then conflict-free -- measured 205 B/clk per CU
// against 113 with f, which leaves them 2-way bank-conflicted -- and f >> 1
// is distinct over rows 0..7 and over rows 8..15, so each half-wave of a V
// transpose read (8 rows x 2 adjacent chunks) covers all 16 chunk positions
// once (177 B/clk).  Otherwise (bf16 D = 64, E4M3 D = 128: 8 chunks) both
// use r mod 8.
template <int D, int ES, int NT = kThreads>
struct Ring {
  static constexpr int RB = D * ES;                  // bytes per row
  static constexpr int CH = RB / 16;                 // 16-byte chunks per row
  static constexpr int SUB = 32;                     // keys per sub-tile
  static constexpr int PART = SUB * RB;              // bytes of K (or V) per sub-tile
  static constexpr int SLOT = 2 * PART;              // K + V
  // sub-tiles in the ring: all of LDS for bf16 with 512-thread workgroups
  // (10), half of it with 256-thread ones (two workgroups per CU: 5); 10 for
  // E4M3 (80 KB) either way: a deeper ring, every slot requested at the
  // start, made the first sub-tiles land later (measured 1-6 % slower calls)
  static constexpr int NS = ES == 1 ? 10 : (160 * 1024 / (kThreads / NT)) / SLOT;
  static constexpr int DPS = 2 * SUB * CH / NT;  // copies per thread per sub-tile
  static constexpr int BYTES = NS * SLOT;
  static_assert((DPS == 1 || DPS % 2 == 0) && (2 * SUB * CH) % NT == 0, "sub-tile split");
  __device__ static int swz_k(int row, int chunk) { return chunk ^ (row & (CH - 1)); }
  __device__ static int swz_v(int row, int chunk) {
    if constexpr (CH == 16) return chunk ^ (((row & 7) << 1) | ((row >> 3) & 1));
    else return chunk ^ (row & (CH - 1));
  }
};

template <int D, int QB, int WR, bool F8, bool PAGED, int NT = kThreads>
__global__ void __launch_bounds__(NT, kThreads / NT) k_attn_mfma(AttnParams p) {
  // F8: keys and values are OCP E4M3 codes (scaled per KV head), widened to
  // bf16 exactly after the LDS reads; everything else is the bf16 kernel
  using KV = std::conditional_t<F8, uint8_t, uint16_t>;
  constexpr int ES = F8 ? 1 : 2;
  using R = Ring<D, ES, NT>;
  constexpr int WK = (NT / PTD_WAVE) / WR;  // key groups: sub-tiles per round
  constexpr int DB = D / 32;                      // 32-wide d blocks (QK^T k-dim)
  constexpr int DT = D / 16;                      // 16-wide d tiles (PV output rows)
  constexpr int PARK_O = WK > 1 ? WR * WK * QB * DT * 64 * 16 : 0;  // parked fragments
  constexpr int PARK_BYTES = PARK_O + (WK > 1 ? WR * WK * QB * 64 * 8 : 0);
  constexpr int SMEM = R::BYTES > PARK_BYTES ? R::BYTES : PARK_BYTES;
  static_assert(R::NS >= 2 * WK, "ring must hold two rounds");
  constexpr int QROWS = 16 * QB * WR;             // query rows of a workgroup
  constexpr int CHQ = D / 8;                      // 16-byte chunks of one
  constexpr int QS = (QROWS * D * 2 + R::SLOT - 1) / R::SLOT;  // ring slots that hold them at first
  static_assert(R::NS - QS >= WK, "round 0 beside the query rows");
  static_assert(R::NS * R::DPS <= 63, "vector-memory counter range");
  __shared__ __attribute__((aligned(16))) unsigned char smem[SMEM];

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int wr = wave % WR;
  const int kg = wave / WR;
  const int l16 = lane & 15;
  const int l4 = lane >> 4;

  // A batch of up to 64 sequences is taken largest first (size = committed
  // keys + tree nodes; ties in index order): the longest workgroups start
  // first and the short ones fill in at the end.  Work item b names the b-th
  // largest sequence; each wave ranks the sizes, lane l holding sequence l's
  // lengths, which then need no second load (85.4 against 86.7 us on 16 sequences
  // of 512-8192 keys).
  const bool by_size = p.B > 1 && p.B <= PTD_WAVE;
  int id;
  logical_block(blockIdx.x, gridDim.x, p.B * p.Hkv, by_size, id);
  const int split = id % p.splits;
  int rest = id / p.splits;
  const int pass = rest % p.passes;
  rest /= p.passes;
  const int g = rest % p.Hkv;
  int b = rest / p.Hkv;
  int n_kv, tl;
  if (by_size) {
    int kvl = 0, tll = 0, nl = -1;
    if (lane < p.B) {  // clamped: an invalid kv_len is reported below, not summed
      kvl = p.kv_len[lane];
      tll = live_nodes(p, lane);
      nl = (kvl < 0 ? -1 : min(kvl, p.L_cap)) + tll;
    }
    int rank = 0;
    for (int j = 0; j < p.B; ++j) {
      const int nj = __builtin_amdgcn_readlane(nl, j);
      rank += (nj > nl || (nj == nl && j < lane)) ? 1 : 0;
    }
    // the ranks of lanes < B are a permutation of 0 .. B-1: one lane hits
    const uint64_t hit = __ballot(lane < p.B && rank == b);
    b = hit ? __builtin_ctzll(hit) : b;
    n_kv = __builtin_amdgcn_readlane(kvl, b);
    tl = __builtin_amdgcn_readlane(tll, b);
  } else {
    n_kv = p.kv_len[b];
    tl = live_nodes(p, b);
  }
  if (n_kv < 0 || n_kv > p.L_cap - tl) {  // (no overflow near the int range)
    if (tid == 0) ptd::report(p.dev_status, PTD_ERR_KV_LEN);
    return;
  }
  const int N = n_kv + tl;
  const int csz = chunk_size(N, p.splits);
  const int start = split * csz;
  const int end = min(N, start + csz);
  // Rows of padding nodes are neither computed nor kept as partials (16
  // sequences of 21-64 live nodes in 64 slots: 86.7 against 104.1 us per call with
  // every slot computed).
  const int pr0 = pass * p.rows_per_pass;
  const int m_live = tl * p.G;
  if (start >= end || pr0 >= m_live) {  // empty split (the combine skips it), or padding rows only
    if (p.splits == 1) {  // zero rows
      const int r0 = pr0, r1 = min(p.M, r0 + p.rows_per_pass);
      for (int x = tid; x < (r1 - r0) * D; x += NT) {
        const int r = r0 + x / D, d = x % D;
        const size_t off = ((static_cast<size_t>(b) * p.T + r / p.G) * p.Hq + g * p.G + r % p.G) * D + d;
        if (p.out_bf16) static_cast<uint16_t*>(p.out)[off] = 0;
        else static_cast<float*>(p.out)[off] = 0.f;
      }
    }
    if constexpr (PAGED) {  // no live node: the page ids of the keys are still checked
      if (pass == 0) {
        const int32_t* pt = p.page_table + static_cast<size_t>(b) * p.max_pages;
        bool bad = false;
        for (int i = (start >> p.page_shift) + tid; start < end && i <= (end - 1) >> p.page_shift; i += NT)
          bad |= static_cast<uint32_t>(pt[i]) >= static_cast<uint32_t>(p.num_pages);
        if (bad) ptd::report(p.dev_status, PTD_ERR_PAGE);
      }
    }
    return;
  }

  const KV* kbase = static_cast<const KV*>(p.k) +
                    (PAGED ? 0 : (static_cast<size_t>(b) * p.Hkv + g) * p.L_cap * D);
  const KV* vbase = static_cast<const KV*>(p.v) +
                    (PAGED ? 0 : (static_cast<size_t>(b) * p.Hkv + g) * p.L_cap * D);
  // paged: the split's first 256 page ids, one per lane and register
  const int first_page = PAGED ? (start >> p.page_shift) : 0;
  uint32_t pg[4] = {0u, 0u, 0u, 0u};
  if constexpr (PAGED) {
    const int npg = ((end - 1) >> p.page_shift) - first_page + 1;
    const int32_t* pt = p.page_table + static_cast<size_t>(b) * p.max_pages + first_page;
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (r * PTD_WAVE + lane < npg) pg[r] = static_cast<uint32_t>(pt[r * PTD_WAVE + lane]);
  }
  const int rowbase = pr0 + wr * 16 * QB;
  const bool wave_live = rowbase < m_live;  // padding waves only copy and sync

  // ---- parent[] entries for deriving ancestor words in-kernel (trees of <= 128
  //      nodes: two per lane)
  const bool small_tree = p.W <= 2;
  const int32_t* pb = p.parent + static_cast<size_t>(b) * p.T;
  int par_lo = lane < p.T ? pb[lane] : -1;
  int par_hi = lane + 64 < p.T ? pb[lane + 64] : -1;
  if constexpr (PAGED) {  // an id out of range is reported and page 0 read instead
    bool bad = false;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if (pg[r] >= static_cast<uint32_t>(p.num_pages)) {
        bad = true;
        pg[r] = 0u;
      }
    }
    if (__any(bad) && tid == 0) ptd::report(p.dev_status, PTD_ERR_PAGE);
  }

  const uint32_t ring = lds_addr(smem);
  // ---- query rows to the ring's last slots, ahead of the first sub-tiles; their
  //      fragments are read once both have landed, then the slots get theirs.
  //      Row r's chunk s lies at position s ^ (r mod CHQ).  (Loads into registers
  //      have to be waited for before the first copy, as the compiler does not count
  //      the copies: 32 heads x 64 rows x 2112 keys with the embedding 20.9 against
  //      20.5 us, batches 0.2-0.5 us a call.  From inline asm, fenced after a later
  //      wait, the compiler takes their registers as written at once and may copy or
  //      reuse them while the data is on its way.)
  {
    constexpr int STEP = NT / CHQ;  // rows per copy (a multiple of CHQ)
    const int row = tid / CHQ;
    const int ch = (tid % CHQ) ^ (row & (CHQ - 1));
    int r = pr0 + row, i = r / p.G, hg = r % p.G;
    const int di = STEP / p.G, dh = STEP % p.G;  // uniform
    const uint16_t* qb0 = static_cast<const uint16_t*>(p.q) +
                          (static_cast<size_t>(b) * p.T * p.Hq + g * p.G) * D + 8 * ch;
#pragma unroll
    for (int u = 0; u < (QROWS + STEP - 1) / STEP; ++u) {
      if (u * STEP + wave * PTD_WAVE / CHQ < QROWS) {  // uniform; rows past the last one re-read it
        const int ic = r < p.M ? i : p.T - 1, hc = r < p.M ? hg : p.G - 1;
        dma16(qb0 + (static_cast<size_t>(ic) * p.Hq + hc) * D,
              ring + (R::NS - QS) * R::SLOT + (u * NT + wave * PTD_WAVE) * 16);
      }
      r += STEP;
      i += di;
      hg += dh;
      if (hg >= p.G) {
        hg -= p.G;
        ++i;
      }
    }
  }

  // ---- sub-tile copies: thread tid moves chunks u*512 + tid of the
  //      sub-tile's 2*32*CH chunks (K rows, then V rows); chunk u of a thread
  //      is K or V for the whole wave (SUB*CH is a multiple of 64)
  uint32_t cp_voff[R::DPS], cp_lds[R::DPS];
  int cp_row[R::DPS], cp_off[R::DPS];
  bool cp_v[R::DPS];
#pragma unroll
  for (int u = 0; u < R::DPS; ++u) {
    const int c = u * NT + tid;
    cp_v[u] = (u * NT + wave * PTD_WAVE) / (R::SUB * R::CH) != 0;
    const int local = c % (R::SUB * R::CH);
    cp_row[u] = local / R::CH;
    cp_off[u] = (cp_v[u] ? R::swz_v(cp_row[u], local % R::CH)
                         : R::swz_k(cp_row[u], local % R::CH)) * (16 / ES);  // elements
    cp_voff[u] = static_cast<uint32_t>((cp_row[u] * D + cp_off[u]) * ES);
    cp_lds[u] = static_cast<uint32_t>((u * NT + wave * PTD_WAVE) * 16);
  }
  // physical page of the split's ti-th page, ti < 256 (staged in pg)
  auto staged_page = [&](int ti) __attribute__((always_inline)) -> uint32_t {
    const uint32_t v0 = __builtin_amdgcn_readlane(pg[0], ti & 63);
    const uint32_t v1 = __builtin_amdgcn_readlane(pg[1], ti & 63);
    const uint32_t v2 = __builtin_amdgcn_readlane(pg[2], ti & 63);
    const uint32_t v3 = __builtin_amdgcn_readlane(pg[3], ti & 63);
    const int k = ti >> 6;
    return k == 0 ? v0 : k == 1 ? v1 : k == 2 ? v2 : v3;
  };
  // element offset of key row `row0` in its page
  auto page_offset = [&](uint32_t phys, int row0) __attribute__((always_inline)) -> size_t {
    return (((static_cast<size_t>(phys) * p.Hkv + g) << p.page_shift) +
            (row0 & ((1 << p.page_shift) - 1))) * D;
  };
  // element offset of key row `row0` (a multiple of 32): contiguous, or in
  // its page (a page holds a multiple of 32 rows, so the sub-tile's 32 rows
  // are consecutive there)
  auto tile_offset = [&](int row0) __attribute__((always_inline)) -> size_t {
    if constexpr (!PAGED) return static_cast<size_t>(row0) * D;
    const int ti = (row0 >> p.page_shift) - first_page;  // uniform
    uint32_t phys;
    if (ti < 4 * PTD_WAVE) {
      phys = staged_page(ti);
    } else {  // beyond the staged ids: a scalar load (checked the same way)
      phys = static_cast<uint32_t>(
          p.page_table[static_cast<size_t>(b) * p.max_pages + (row0 >> p.page_shift)]);
      if (phys >= static_cast<uint32_t>(p.num_pages)) {
        if (tid == 0) ptd::report(p.dev_status, PTD_ERR_PAGE);
        phys = 0u;
      }
    }
    return page_offset(phys, row0);
  };
  // copy sub-tile t (keys start + 32t ..) into ring slot `slot`
  auto issue = [&](int t, int slot) __attribute__((always_inline)) {
    const uint32_t slot_lds = ring + slot * R::SLOT;
    const int row0 = start + t * R::SUB;
    const size_t tile = tile_offset(row0);
    if (row0 + R::SUB <= N) {  // whole sub-tile inside the keys: scalar base
      if constexpr (R::DPS == 1) {
        dma16_s((cp_v[0] ? vbase : kbase) + tile, cp_voff[0], slot_lds + cp_lds[0]);
      } else {
#pragma unroll
        for (int u = 0; u < R::DPS; u += 2)
          ptd::dma16_s2((cp_v[u] ? vbase : kbase) + tile, cp_voff[u], slot_lds + cp_lds[u],
                        (cp_v[u + 1] ? vbase : kbase) + tile, cp_voff[u + 1], slot_lds + cp_lds[u + 1]);
      }
    } else {  // last sub-tile: rows past the keys re-read the last key
#pragma unroll
      for (int u = 0; u < R::DPS; ++u) {
        const int grow = min(row0 + cp_row[u], N - 1);
        dma16((cp_v[u] ? vbase : kbase) + tile + static_cast<size_t>(grow - row0) * D + cp_off[u],
              slot_lds + cp_lds[u]);
      }
    }
  };

  const int ntiles = (end - start + R::SUB - 1) / R::SUB;
  const int nrounds = (ntiles + WK - 1) / WK;
  const int ninit = min(ntiles, R::NS);

  // query fragments (B operand of S^T = K Q^T: lane holds Q[row l16][d = 32*db +
  // 8*l4 .. +8]), read once they have landed
  bf16x8 qf[QB][DB];

  // per-lane LDS byte offsets inside a sub-tile (the row's swizzle is the
  // same for both 16-row halves, which therefore differ by a constant)
  int koff[DB], voff[DT];
  if constexpr (F8) {
    // K: lane (l16, l4) reads the 8 bytes d = 32*db + 8*l4 .. of key l16.
    // V: source lane l16 = 2j + h of group l4 points at key slot j's row
    // (keys 4*l4 + j, j < 4, and 16 + 4*l4 + j - 4), bytes 16*dt + 8h ..;
    // the transpose read gives lane l16 the 8 keys' values at d = 16*dt + l16.
#pragma unroll
    for (int db = 0; db < DB; ++db)
      koff[db] = l16 * R::RB + R::swz_k(l16, 2 * db + (l4 >> 1)) * 16 + (l4 & 1) * 8;
    const int j = l16 >> 1, h = l16 & 1;
    const int key0 = j < 4 ? 4 * l4 + j : 16 + 4 * l4 + (j - 4);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) voff[dt] = key0 * R::RB + R::swz_v(key0, dt) * 16 + h * 8;
  } else {
#pragma unroll
    for (int db = 0; db < DB; ++db)
      koff[db] = l16 * R::RB + R::swz_k(l16, db * 4 + l4) * 16;
    const int tj = l16 >> 2, tq = l16 & 3;
    const int key0 = 4 * l4 + tj;  // this lane's source key for the transpose reads
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
      voff[dt] = key0 * R::RB + R::swz_v(key0, 2 * dt + (tq >> 1)) * 16 + (tq & 1) * 8;
  }

  struct Tile {
    f32x4 s[2][QB];
  };
  struct KFrag {
    bf16x8 k[DB][2];
  };
  // K fragments of the sub-tile in `slot` (A operand: 16 keys x 32 d)
  auto read_k = [&](int slot) __attribute__((always_inline)) -> KFrag {
    KFrag f;
    const unsigned char* ks = smem + slot * R::SLOT;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        if constexpr (F8)
          f.k[db][kb] = e4m3x8_to_bf16(*reinterpret_cast<const u32x2*>(ks + kb * 16 * R::RB + koff[db]));
        else
          f.k[db][kb] = __builtin_bit_cast(
              bf16x8, *reinterpret_cast<const u32x4*>(ks + kb * 16 * R::RB + koff[db]));
      }
    return f;
  };
  // S^T (keys x queries) = K Q^T; lane: query l16, keys 16*kb + 4*l4 + e
  auto qk = [&](const KFrag& f) __attribute__((always_inline)) -> Tile {
    Tile x;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) x.s[kb][qb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
          x.s[kb][qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.k[db][kb], qf[qb][db], x.s[kb][qb], 0, 0, 0);
    return x;
  };
  // V^T fragments (A operand of O^T += V^T P^T).  K-slot j of lane group l4
  // is key 4*l4 + j (j < 4) or 16 + 4*l4 + (j - 4), matching the S^T layout;
  // source lane 4*j + q of a 16-lane group points at V[key_j][16*dt + 4q],
  // and lane i of the group receives V[key_0..3][16*dt + i].
  struct VFrag {
    bf16x8 v[DT];
  };
  auto read_v = [&](int slot) __attribute__((always_inline)) -> VFrag {
    VFrag f;
    const unsigned char* vs = smem + slot * R::SLOT + R::PART;
    if constexpr (F8) {
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) f.v[dt] = e4m3x8_to_bf16(lds_read_tr8(vs + voff[dt]));
      return f;
    }
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      const i16x4 lo = lds_read_tr16(vs + voff[dt]);
      const i16x4 hi = lds_read_tr16(vs + 16 * R::RB + voff[dt]);
      const u32x2 l2 = __builtin_bit_cast(u32x2, lo);
      const u32x2 h2 = __builtin_bit_cast(u32x2, hi);
      const u32x4 vv = {l2[0], l2[1], h2[0], h2[1]};
      f.v[dt] = __builtin_bit_cast(bf16x8, vv);
    }
    return f;
  };

  // ---- scores of keys past the chunk end, or of tree keys that are not
  //      ancestors, become -inf.  The ancestor words of the rows' nodes are
  //      held from a sub-tile to the next ones (128 nodes: word mbase and the
  //      one after it).  For trees of <= 128 nodes they are derived here at the
  //      first sub-tile with tree keys (only the last few of a sequence):
  //      every lane follows the parent chains of its rows' nodes (parent[a]
  //      read from lane a % 64 by shuffles, all lanes active); each step moves
  //      to a lower index, so 128 steps end every walk.  Larger trees read the
  //      mask pass's rows, two words at a time: the compiler's wait for such a
  //      load also waits for the ring copies in flight (256 nodes x 2 sequences
  //      of 1000-4096 keys: 60.2 us per call against 68.0 with a load per key).
  // first sub-tile reaching past the committed keys or the chunk end
  const int t_mask0 = max(0, (min(n_kv, end) - start) / R::SUB);
  uint64_t mw0[QB], mw1[QB];
  int mbase = -1;  // no words held
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) mw0[qb] = mw1[qb] = 0ull;
  auto node_of = [&](int qb) __attribute__((always_inline)) {
    return min(rowbase + qb * 16 + l16, p.M - 1) / p.G;
  };
  auto walk_words = [&]() __attribute__((always_inline)) {
    int a[QB];  // padding nodes see no tree keys (and their parents are not read)
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      const int node = node_of(qb);
      a[qb] = node < tl ? node : -1;
      mw0[qb] = mw1[qb] = 0ull;
    }
    for (int step = 0; step < 128; ++step) {
      bool live = false;
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) live |= a[qb] >= 0;
      if (!__any(live)) break;
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) {
        const int xa = a[qb];
        const uint64_t bit = 1ull << (xa & 63);  // branchless: no indexed word pair
        mw0[qb] |= (xa >= 0 && xa < 64) ? bit : 0ull;
        mw1[qb] |= (xa >= 64) ? bit : 0ull;
        const int plo = __shfl(par_lo, xa & 63, PTD_WAVE);
        const int phi = __shfl(par_hi, xa & 63, PTD_WAVE);
        int nx = xa >= 64 ? phi : plo;
        if (xa < 0) {
          nx = -1;
        } else if (nx < -1 || nx >= xa) {  // not topological
          ptd::report(p.dev_status, PTD_ERR_BAD_TREE);
          nx = -1;
        }
        a[qb] = nx;
      }
    }
  };
  auto mask_tile = [&](Tile& x, int t) __attribute__((always_inline)) {
    if (t < t_mask0) return;
    const int abs0 = start + t * R::SUB;
    const int off = abs0 - n_kv;  // node of the sub-tile's first key (uniform, > -32 with tree keys)
    const int rem = end - abs0;   // keys before the chunk end
    const uint32_t in_chunk = rem >= 32 ? ~0u : (1u << rem) - 1u;
    uint32_t vis[QB];  // bit k: key abs0 + k is visible to the lane's row
    if (off > -R::SUB) {
      const int w = max(off, 0) >> 6;
      if (small_tree) {
        if (mbase < 0) {
          walk_words();
          mbase = 0;
        }
      } else if (mbase < 0 || max(off, 0) + R::SUB > (mbase + 2) * 64) {
        mbase = w;
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
          const uint64_t* row = p.mask + (static_cast<size_t>(b) * p.T + node_of(qb)) * p.W;
          mw0[qb] = w < p.W ? row[w] : 0ull;
          mw1[qb] = w + 1 < p.W ? row[w + 1] : 0ull;
        }
        // waited for here: a load pending at the steady loop would make the
        // compiler wait for every ring copy inside it
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) asm volatile("" : "+v"(mw0[qb]), "+v"(mw1[qb]));
      }
      const int s = off - 64 * mbase;  // < 128
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) {
        if (s < 0) vis[qb] = (static_cast<uint32_t>(mw0[qb]) << -s) | ((1u << -s) - 1u);
        else if (s == 0) vis[qb] = static_cast<uint32_t>(mw0[qb]);
        else if (s < 64) vis[qb] = static_cast<uint32_t>((mw0[qb] >> s) | (mw1[qb] << (64 - s)));
        else vis[qb] = static_cast<uint32_t>(mw1[qb] >> (s - 64));
      }
    } else {  // committed keys only
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) vis[qb] = ~0u;
    }
    // visibility as selects only: per-element branches writing the tile
    // through this lambda's reference were miscompiled
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      const uint32_t v = (vis[qb] & in_chunk) >> (4 * l4);
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          x.s[kb][qb][e] = (v & (1u << (16 * kb + e))) != 0 ? x.s[kb][qb][e] : -INFINITY;
    }
  };

  // ---- online softmax state.  Scores become p = 2^(s*c - m*c) against a
  //      reference maximum m per query row that moves lazily: while no p of a
  //      sub-tile exceeds 2^16, O and l stay far inside the fp32 range and m
  //      is kept.  Otherwise (the first keys a row sees, m still at its start
  //      value, or a score well above m) the rows' maxima are formed, m moves
  //      up to them, O and l are rescaled and the sub-tile's p are recomputed.
  //      The row sums l run on the matrix cores: an MFMA of the bf16 P
  //      fragment with an all-ones A operand gives every output row the sums
  //      of P's columns over the 32 keys, so each lane holds its query
  //      column's l with no cross-lane reduction (two MFMAs per sub-tile
  //      against about thirty vector instructions for dot products and
  //      cross-lane sums).
  f32x4 o[QB][DT];
  float m[QB], nmc[QB];
  f32x4 ls[QB];  // row sums of p (all four elements: the lane's query column)
  // score scale in the exp2 domain; 8-bit keys carry their head's scale
  const float c = F8 && p.k_scale ? p.c * p.k_scale[g] : p.c;
  const float vsc = F8 && p.v_scale ? p.v_scale[g] : 1.0f;  // value scale
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    m[qb] = kNegBig;
    nmc[qb] = -kNegBig * c;
    ls[qb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) o[qb][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  // exponentials of a tile, and the largest of each lane's eight
  auto exp_tile = [&](const Tile& x, float (&pv)[QB][8], float (&pm)[QB]) __attribute__((always_inline)) {
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        pv[qb][e] = __builtin_amdgcn_exp2f(fmaf(x.s[0][qb][e], c, nmc[qb]));
        pv[qb][4 + e] = __builtin_amdgcn_exp2f(fmaf(x.s[1][qb][e], c, nmc[qb]));
      }
      pm[qb] = fmaxf(fmaxf(fmaxf(pv[qb][0], pv[qb][1]), fmaxf(pv[qb][2], pv[qb][3])),
                     fmaxf(fmaxf(pv[qb][4], pv[qb][5]), fmaxf(pv[qb][6], pv[qb][7])));
    }
  };
  // bf16 ones: A operand of the row-sum MFMA (every output row = the sum of
  // the B operand's column over the 32 keys)
  const bf16x8 ones8 = __builtin_bit_cast(bf16x8, u32x4{0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u});
  // rare: move the reference of rows whose maximum passed it (uniform over
  // the row's four lanes).  Every lane runs the same instructions (a factor
  // of 1 where the reference stays): rescaling accumulators under a per-lane
  // branch returned wrong row sums in some builds.
  auto move_ref = [&](const Tile& x) __attribute__((always_inline)) {
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      float mx = fmaxf(fmaxf(fmaxf(x.s[0][qb][0], x.s[0][qb][1]), fmaxf(x.s[0][qb][2], x.s[0][qb][3])),
                       fmaxf(fmaxf(x.s[1][qb][0], x.s[1][qb][1]), fmaxf(x.s[1][qb][2], x.s[1][qb][3])));
      mx = max_xor32(max_xor16(mx));
      const bool up = mx > m[qb];
      const float alpha = up ? __builtin_amdgcn_exp2f((m[qb] - mx) * c) : 1.0f;  // 0 for the first keys
      m[qb] = up ? mx : m[qb];
      nmc[qb] = up ? -mx * c : nmc[qb];
      ls[qb] *= alpha;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) o[qb][dt] *= alpha;
    }
  };
  // p of a tile as bf16 MFMA operands (B of O^T += V^T P^T: lane holds its
  // query column's 8 keys); for precise query blocks also the rounding
  // residue p - bf16(p)
  struct PFrag {
    bf16x8 hi[QB], lo[QB];
  };
  auto pv_acc = [&](const VFrag& v, const PFrag& f, unsigned precise) __attribute__((always_inline)) {
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int qb = 0; qb < QB; ++qb)
        o[qb][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v.v[dt], f.hi[qb], o[qb][dt], 0, 0, 0);
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) ls[qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones8, f.hi[qb], ls[qb], 0, 0, 0);
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
      if (precise & (1u << qb)) {
        ls[qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones8, f.lo[qb], ls[qb], 0, 0, 0);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
          o[qb][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v.v[dt], f.lo[qb], o[qb][dt], 0, 0, 0);
      }
  };

  // ---- rounds.  Round rd holds sub-tiles rd*WK .. rd*WK + WK - 1 (wave kg
  //      takes rd*WK + kg).  Software pipeline (PIPE): during round rd a wave
  //      issues the QK^T MFMAs of its round rd + 1 sub-tile interleaved with
  //      the softmax of its round rd sub-tile (scores kept in registers from
  //      the round before), then the PV MFMAs of round rd.  Round rd thus
  //      reads K of round rd + 1 and V of round rd, the data of round rd + 1
  //      is waited for at the barrier of round rd, and the slots of round
  //      rd - 1 are free there and refilled right away.  Round rd + 1's data
  //      is then issued by round rd - 1, which needs 3*WK ring slots; with
  //      more key groups a round computes its own sub-tile start to end.
  //      The denominator adds the same bf16 p that enter O, so that O is
  //      the exact average of V under the rounded weights.  A query block
  //      of a tile in which some p exceeds kPreciseFrac of its row's sum so
  //      far (this wave's keys, from the row-sum accumulator)
  //      carries p as bf16 hi + lo (residue at most 2^-16 p instead of
  //      2^-8 p): every key carried as plain bf16 then weighs at most
  //      kPreciseFrac of its row's final sum, so the 2^-8 relative rounding
  //      of a dominant key, or of a few large ones, never reaches O.
  constexpr bool PIPE = 3 * WK <= R::NS;
  static_assert((2 + (PIPE ? 1 : 0)) * WK <= R::NS, "round data issued one round ahead");
  // bf16 p of scores x (exponentials pv and lane maxima pm computed);
  // returns the mask of precise query blocks (residues in f.lo)
  auto to_p = [&](const Tile& x, float (&pv)[QB][8], float (&pm)[QB], PFrag& f)
      __attribute__((always_inline)) -> unsigned {
    bool over = false;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) over |= !(pm[qb] <= 65536.0f);
    if (__any(over)) {
      move_ref(x);
      exp_tile(x, pv, pm);
    }
    unsigned pmask = 0;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
      pmask |= __any(!(pm[qb] <= p.precise * ls[qb][0])) ? (1u << qb) : 0u;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      const bool precise = pmask & (1u << qb);
      u32x4 ph, pl;
#pragma unroll
      for (int w = 0; w < 4; ++w) ph[w] = ptd::cvt_pk_bf16(pv[qb][2 * w], pv[qb][2 * w + 1]);
      f.hi[qb] = __builtin_bit_cast(bf16x8, ph);
      if (precise) {
#pragma unroll
        for (int w = 0; w < 4; ++w)
          pl[w] = ptd::cvt_pk_bf16(pv[qb][2 * w] - static_cast<float>(f.hi[qb][2 * w]),
                                   pv[qb][2 * w + 1] - static_cast<float>(f.hi[qb][2 * w + 1]));
        f.lo[qb] = __builtin_bit_cast(bf16x8, pl);
      }
    }
    return pmask;
  };

  const int nfirst = min(ninit, R::NS - QS);
  for (int t = 0; t < nfirst; ++t) issue(t, t);
  wait_vmcnt_le((nfirst - min(ntiles, WK)) * R::DPS);  // query rows and round 0 landed
  lds_barrier();
#pragma unroll
  for (int qb = 0; qb < QB; ++qb)
#pragma unroll
    for (int db = 0; db < DB; ++db)
      qf[qb][db] = *reinterpret_cast<const bf16x8*>(
          smem + (R::NS - QS) * R::SLOT + ((wr * QB + qb) * 16 + l16) * D * 2 +
          ((db * 4 + l4) ^ (l16 & (CHQ - 1))) * 16);
  if (ninit > nfirst) {  // uniform
    lds_barrier();  // every wave has its fragments
    for (int t = nfirst; t < ninit; ++t) issue(t, t);
  }

  // rounds whose wait count is the steady-state constant: every refill so far
  // issued in full (R::NS + (rd - 1) * WK <= ntiles)
  const int steady_end = ntiles >= R::NS ? (ntiles - R::NS) / WK + 1 : -1;
  int cs = kg;  // ring slot of this wave's sub-tile of the current round
  int rs = 0;   // slot refilled next (round rd - 1's slots, in order)
  Tile sc;      // PIPE: scores of the current round's sub-tile
  if (PIPE && wave_live && kg < ntiles) {
    sc = qk(read_k(cs));
    mask_tile(sc, kg);
  }
  // a round in general: waits by the count of copies issued so far, refills
  // (whole or last sub-tiles, contiguous or paged caches), masked sub-tiles
  auto round = [&](int rd) __attribute__((always_inline)) {
      const bool do_wait = PIPE ? rd + 1 < nrounds : rd >= 1;
      if (do_wait) {
        if (rd >= 1 && rd <= steady_end) {
          wait_vmcnt<(R::NS - (2 + (PIPE ? 1 : 0)) * WK) * R::DPS>();
        } else {
          const int issued = min(ntiles, R::NS + max(0, rd - 1) * WK);
          const int needed = min(ntiles, (rd + 1 + (PIPE ? 1 : 0)) * WK);
          wait_vmcnt_le((issued - needed) * R::DPS);
        }
        lds_barrier();
        if (rd >= 1) {
#pragma unroll
          for (int w = 0; w < WK; ++w) {
            const int tt = R::NS + (rd - 1) * WK + w;
            if (tt < ntiles) issue(tt, rs);
            rs = rs + 1 == R::NS ? 0 : rs + 1;
          }
        }
      }
      int ns = cs + WK;
      if (ns >= R::NS) ns -= R::NS;
      const int j = rd * WK + kg;
      if (wave_live && j < ntiles) {
        float pv[QB][8], pm[QB];
        if constexpr (PIPE) {
          // next K reads in flight while this sub-tile's exponentials run (they
          // overlap the previous round's PV MFMAs, still executing); then the
          // next QK^T and this PV back to back on the matrix cores.  After the
          // wave's last sub-tile the next-tile QK^T works on whatever the slot
          // holds and its result is dropped: one code path keeps the register
          // allocation of this loop within the two-waves-per-SIMD budget.
          const KFrag kf = read_k(ns);
          exp_tile(sc, pv, pm);
          PFrag pf;
          const unsigned precise = to_p(sc, pv, pm, pf);
          Tile sn = qk(kf);
          const VFrag vf = read_v(cs);
          pv_acc(vf, pf, precise);
          if (j + WK < ntiles) mask_tile(sn, j + WK);
          sc = sn;
        } else {
          sc = qk(read_k(cs));
          mask_tile(sc, j);
          const VFrag vf = read_v(cs);
          exp_tile(sc, pv, pm);
          PFrag pf;
          const unsigned precise = to_p(sc, pv, pm, pf);
          pv_acc(vf, pf, precise);
        }
      }
      cs = ns;
  };
  // Steady rounds: every refill of the round is a whole sub-tile below t_mask0, so this round's and the next round's
  // sub-tiles need no masking either; the wait count is the constant, the
  // tile address scalar arithmetic, and the general round's tests drop out
  // (with and without the software pipeline; without it, 34.9 against 36.7 us
  // per call on 40 heads x 96 rows x 4192 keys).
  // The scalar instructions of a round are issued by the CU's one scalar unit
  // for every wave, and the two waves of a SIMD reach the refills together:
  // measured on 8 KV heads x 256 rows x 32832 keys, 70.7 against 76.0 us per
  // call; on ragged-16, 156.2 against 171.2.  A steady round also splits the
  // hi + lo P of the general round: the bf16 P and its PV and row-sum MFMAs
  // always, the residues and their MFMAs after them in a rarely taken branch,
  // so the main path is one block the scheduling groups below can interleave
  // (the precise test still reads the row sums before this sub-tile, and
  // every accumulator receives hi before lo as in the general round).
  // Paged caches: a refill's page id is one of the 256 staged in registers
  // (scalar lane reads); beyond those the general round reads the table
  // (16 sequences of 512-8192 keys on 64-row pages: 114.3 against 121.2 us per
  // call with general rounds only; 6 of 1024-16384 on E4M3 pages 69.6 against 71.6).
  int t_steady = t_mask0;
  if constexpr (PAGED) {
    const long long staged = (static_cast<long long>(first_page + 4 * PTD_WAVE) << p.page_shift) - start;
    t_steady = static_cast<int>(min(static_cast<long long>(t_mask0), staged / R::SUB));
  }
  const int steady_hi = t_steady >= R::NS + WK ? (t_steady - R::NS - WK) / WK + 1 : 0;
  auto round_steady = [&](int rd) __attribute__((always_inline)) {
    wait_vmcnt<(R::NS - (2 + (PIPE ? 1 : 0)) * WK) * R::DPS>();
    lds_barrier();
#pragma unroll
    for (int w = 0; w < WK; ++w) {
      const int tt = R::NS + (rd - 1) * WK + w;
      const int row0 = start + tt * R::SUB;
      size_t tile;
      if constexpr (PAGED) tile = page_offset(staged_page((row0 >> p.page_shift) - first_page), row0);
      else tile = static_cast<size_t>(row0) * D;
      const uint32_t slot_lds = ring + rs * R::SLOT;
      if constexpr (R::DPS == 1) {
        dma16_s((cp_v[0] ? vbase : kbase) + tile, cp_voff[0], slot_lds + cp_lds[0]);
      } else {
#pragma unroll
        for (int u = 0; u < R::DPS; u += 2)
          ptd::dma16_s2((cp_v[u] ? vbase : kbase) + tile, cp_voff[u], slot_lds + cp_lds[u],
                        (cp_v[u + 1] ? vbase : kbase) + tile, cp_voff[u + 1],
                        slot_lds + cp_lds[u + 1]);
      }
      rs = rs + 1 == R::NS ? 0 : rs + 1;
    }
    int ns = cs + WK;
    if (ns >= R::NS) ns -= R::NS;
    if constexpr (PIPE) {
      if (wave_live) {
        float pv[QB][8], pm[QB];
        const KFrag kf = read_k(ns);
        exp_tile(sc, pv, pm);
        Tile sn = qk(kf);
        // the K reads, a few exponentials, then one QK^T MFMA per three
        // vector instructions (scheduling groups: 0x100 LDS reads, 0x002
        // vector ALU, 0x008 MFMA)
        __builtin_amdgcn_sched_group_barrier(0x100, 2 * DB, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, 6, 0);
#pragma unroll
        for (int i = 0; i < 2 * QB * DB; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);
        }
        bool over = false;
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) over |= !(pm[qb] <= 65536.0f);
        if (__any(over)) {
          move_ref(sc);
          exp_tile(sc, pv, pm);
        }
        unsigned pmask = 0;
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
          pmask |= __any(!(pm[qb] <= p.precise * ls[qb][0])) ? (1u << qb) : 0u;
        PFrag pf;
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
          u32x4 ph;
#pragma unroll
          for (int w = 0; w < 4; ++w) ph[w] = ptd::cvt_pk_bf16(pv[qb][2 * w], pv[qb][2 * w + 1]);
          pf.hi[qb] = __builtin_bit_cast(bf16x8, ph);
        }
        const VFrag vf = read_v(cs);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int qb = 0; qb < QB; ++qb)
            o[qb][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf.v[dt], pf.hi[qb], o[qb][dt], 0, 0, 0);
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) ls[qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones8, pf.hi[qb], ls[qb], 0, 0, 0);
        // the V reads, then one PV MFMA per two vector instructions
        __builtin_amdgcn_sched_group_barrier(0x100, 2 * DT, 1);
#pragma unroll
        for (int i = 0; i < DT * QB; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 1);
          __builtin_amdgcn_sched_group_barrier(0x002, 2, 1);
        }
        if (pmask) {
#pragma unroll
          for (int qb = 0; qb < QB; ++qb)
            if (pmask & (1u << qb)) {
              u32x4 pl;
#pragma unroll
              for (int w = 0; w < 4; ++w)
                pl[w] = ptd::cvt_pk_bf16(pv[qb][2 * w] - static_cast<float>(pf.hi[qb][2 * w]),
                                         pv[qb][2 * w + 1] - static_cast<float>(pf.hi[qb][2 * w + 1]));
              pf.lo[qb] = __builtin_bit_cast(bf16x8, pl);
              ls[qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones8, pf.lo[qb], ls[qb], 0, 0, 0);
#pragma unroll
              for (int dt = 0; dt < DT; ++dt)
                o[qb][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf.v[dt], pf.lo[qb], o[qb][dt], 0, 0, 0);
            }
        }
        sc = sn;
      }
    } else {
      if (wave_live) {
        float pv[QB][8], pm[QB];
        sc = qk(read_k(cs));
        const VFrag vf = read_v(cs);
        exp_tile(sc, pv, pm);
        PFrag pf;
        const unsigned precise = to_p(sc, pv, pm, pf);
        pv_acc(vf, pf, precise);
      }
    }
    cs = ns;
  };
  int rd0 = 0;
  if (steady_hi >= 1) {
    round(0);
    for (int rd = 1; rd <= steady_hi; ++rd) round_steady(rd);
    rd0 = steady_hi + 1;
    mbase = -1;  // no masked sub-tile yet: no words live over the steady rounds
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) mw0[qb] = mw1[qb] = 0ull;
  }
  for (int rd = rd0; rd < nrounds; ++rd) round(rd);
  wait_vmcnt<0>();
  lds_barrier();  // every copy landed and every wave is done with the ring


  // ---- softmax denominators (each lane: its query column's)
  float lsum[QB];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) lsum[qb] = ls[qb][0];

  // ---- epilogue.  The key groups of a row group hold their fragments in the
  //      same lane layout (lane: query column l16, d = 16*dt + 4*l4 + 0..3), so
  //      the merge is lane-local: every wave parks its fragments and (m, l)
  //      per column in LDS, then wave (wr, kg) merges the key groups (fixed
  //      order) for d-tiles [kg*DPW, (kg+1)*DPW) of its row group and stores
  //      them.  With one key group the fragments are stored directly.
  constexpr int DPW = DT / WK;  // d-tiles merged and stored per wave
  static_assert(DT % WK == 0, "d-tiles per wave");
  const bool all_rows = rowbase + 16 * QB <= p.M;  // uniform: the common case
  auto store_tile = [&](int qb, int dt, f32x4 acc, float mc, float den) {
    const int r = rowbase + qb * 16 + l16;
    if (!all_rows && r >= p.M) return;
    if (p.splits == 1) {
      const int i = r / p.G, hg = r % p.G;
      const size_t off = ((static_cast<size_t>(b) * p.T + i) * p.Hq + g * p.G + hg) * D +
                         16 * dt + 4 * l4;
      const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
      const f32x4 v = i < tl ? acc * (vsc / den) : zero;
      if (p.out_bf16) {
        const u32x2 w2 = {ptd::cvt_pk_bf16(v[0], v[1]), ptd::cvt_pk_bf16(v[2], v[3])};
        *reinterpret_cast<u32x2*>(static_cast<uint16_t*>(p.out) + off) = w2;
      } else {
        *reinterpret_cast<f32x4*>(static_cast<float*>(p.out) + off) = v;
      }
    } else if (r < m_live) {
      const size_t prow = ((static_cast<size_t>(split) * p.B + b) * p.Hkv + g) * p.M + r;
      *reinterpret_cast<f32x4*>(p.part_o + prow * D + 16 * dt + 4 * l4) = F8 ? acc * vsc : acc;
      if (dt == 0 && l4 == 0) p.part_ml[prow] = make_float2(mc, den);
    }
  };
  // waves of padding rows write their zeros, where the output is written here
  const bool wave_stores = wave_live || (rowbase < p.M && p.splits == 1);
  if constexpr (WK == 1) {
    if (!wave_stores) return;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) store_tile(qb, dt, o[qb][dt], m[qb] * c, lsum[qb]);
  } else {
    f32x4* so = reinterpret_cast<f32x4*>(smem);  // [WR][WK][QB][DT][64]
    float2* sml = reinterpret_cast<float2*>(smem + PARK_O);  // [WR][WK][QB][64]
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) so[(((wr * WK + kg) * QB + qb) * DT + dt) * 64 + lane] = o[qb][dt];
      sml[((wr * WK + kg) * QB + qb) * 64 + lane] = make_float2(m[qb], lsum[qb]);
    }
    lds_barrier();
    if (!wave_stores) return;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      float mk[WK], w[WK];
      float mm = kNegBig, den = 0.f;
#pragma unroll
      for (int k2 = 0; k2 < WK; ++k2) {
        mk[k2] = sml[((wr * WK + k2) * QB + qb) * 64 + lane].x;
        mm = fmaxf(mm, mk[k2]);
      }
#pragma unroll
      for (int k2 = 0; k2 < WK; ++k2) {
        w[k2] = __builtin_amdgcn_exp2f((mk[k2] - mm) * c);
        den += w[k2] * sml[((wr * WK + k2) * QB + qb) * 64 + lane].y;
      }
#pragma unroll
      for (int j = 0; j < DPW; ++j) {
        const int dt = kg * DPW + j;
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k2 = 0; k2 < WK; ++k2) acc += so[(((wr * WK + k2) * QB + qb) * DT + dt) * 64 + lane] * w[k2];
        store_tile(qb, dt, acc, mm * c, den);
      }
    }
  }
}

// ===========================================================================
// split-KV combine: out = sum_s w_s O_s / sum_s w_s l_s, w_s = 2^(mc_s - max mc),
// one thread per (b, g, row, 4 columns), online in the split index (fixed
// order, so the result is deterministic).  A workgroup covers 256 / (D/4)
// consecutive rows of one (b, g): everything per (b, g) is uniform (scalar
// loads and arithmetic) and a thread's row and columns are shifts of its id.
// ===========================================================================
template <int D, int U, bool F32>
__global__ void __launch_bounds__(256) k_attn_combine(AttnParams p) {
  // partial maxima are in the exp2 domain, or (fp32 path) scores as they are
  auto expo = [](float x) __attribute__((always_inline)) {
    return F32 ? expf(x) : __builtin_amdgcn_exp2f(x);
  };
  constexpr int D4 = D / 4;
  constexpr int RPB = 256 / D4;  // rows per workgroup
  const int nrb = (p.M + RPB - 1) / RPB;
  const int bg = static_cast<int>(blockIdx.x) / nrb;  // uniform
  const int rb = static_cast<int>(blockIdx.x) - bg * nrb;
  const int b = bg / p.Hkv;
  const int g = bg - b * p.Hkv;
  const int d4 = threadIdx.x % D4;
  const int r = rb * RPB + static_cast<int>(threadIdx.x) / D4;
  if (r >= p.M) return;
  const int i = r / p.G, hg = r % p.G;
  auto store = [&](const f32x4& v) __attribute__((always_inline)) {
    const size_t off = ((static_cast<size_t>(b) * p.T + i) * p.Hq + g * p.G + hg) * D + d4 * 4;
    if (p.out_bf16) {
      const u32x2 w = {ptd::cvt_pk_bf16(v[0], v[1]), ptd::cvt_pk_bf16(v[2], v[3])};
      *reinterpret_cast<u32x2*>(static_cast<uint16_t*>(p.out) + off) = w;
    } else {
      *reinterpret_cast<f32x4*>(static_cast<float*>(p.out) + off) = v;
    }
  };
  const int n_kv = p.kv_len[b];
  const int tl = live_nodes(p, b);
  const bool valid = n_kv >= 0 && n_kv <= p.L_cap - tl;  // else reported by the attention kernel
  if (p.tree_len && i >= tl) {  // padding nodes: zero, and no partials to read
    if (valid) store(f32x4{0.f, 0.f, 0.f, 0.f});
    return;
  }
  // The partials are loaded, U splits at a time, without waiting for kv_len
  // (the workspace holds all p.splits of them); the updates by empty splits,
  // whose partials were never written, are discarded with selects.
  const size_t stride = static_cast<size_t>(p.B) * p.Hkv * p.M;
  const size_t row0 = (static_cast<size_t>(b) * p.Hkv + g) * p.M + r;
  float2 ml[U];
  f32x4 ov[U];
  auto load_group = [&](int s0) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const size_t pr = row0 + static_cast<size_t>(min(s0 + u, p.splits - 1)) * stride;
      ml[u] = p.part_ml[pr];
      ov[u] = *reinterpret_cast<const f32x4*>(p.part_o + pr * D + d4 * 4);
    }
  };
  load_group(0);
  const int N = valid ? n_kv + tl : 1;
  const int csz = chunk_size(max(N, 1), p.splits);
  const int nsp = (N + csz - 1) / csz;  // non-empty splits
  float mrun = kNegBig, den = 0.f;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  auto merge_group = [&](int s0) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool live = s0 + u < nsp;
      const float mn = fmaxf(mrun, ml[u].x);
      const float a = expo(mrun - mn);
      const float w = expo(ml[u].x - mn);
      const f32x4 na = acc * a + ov[u] * w;
      den = live ? den * a + w * ml[u].y : den;
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] = live ? na[e] : acc[e];
      mrun = live ? mn : mrun;
    }
  };
  merge_group(0);  // the first group outside the loop: its loads stay ahead of every wait
  for (int s0 = U; s0 < nsp; s0 += U) {
    load_group(s0);
    merge_group(s0);
  }
  if (valid) store(acc * (1.0f / den));
}

// ===========================================================================
// fp32 path: v_mfma_f32_16x16x4_f32 (fp32 products and sums).  One workgroup of
// 8 waves per (b, g, 16 query rows, KV split); wave w takes the 16-key tiles
// w, w + 8, .. of the split with a softmax state of its own, and the states
// merge through LDS at the end.
//   S^T = K Q^T per tile: lane (l16, l4) holds K[key l16][16 j + 4 l4 + e] and
//   Q[row l16][same], one 16-byte load each per 16 columns; the MFMA of (j, e)
//   contracts the columns 16 j + 4 l4 + e over the four lane groups.  The lane
//   then owns scores of query l16 and keys 4 l4 + e.
//   O^T += V^T P^T: the MFMA of step e contracts the keys 4 l4 + e, whose p the
//   lane owns already; its A operand for the columns {64 h + 4 i + f} is element
//   f of the 16 bytes V[4 l4 + e][64 h + 4 l16 ..].  No operand passes LDS.
// The next tile's K and this tile's V load while the scores are formed.  Bound by
// latency at the sizes of a reference configuration (2 heads x 16 rows x 144
// keys: 7.9 us for the kernel; one workgroup of vector dot products per (b, g, 32
// rows), one key per lane, took 37.6 and a mask pass before it 1.8; 4 heads x 64
// rows x 576 keys x 128 columns, a whole step of it: 33 against 321 us).
// ===========================================================================
constexpr int kF32Threads = 512;
constexpr int kF32Waves = kF32Threads / PTD_WAVE;
constexpr int kF32Rows = 16;
constexpr int kF32Keys = 16;

// Ancestor words (nodes 0-63, 64-127) of a node of a tree of up to 128 nodes:
// lane x of the wave holds parent[x] and parent[x + 64] (-1 past the tree).
// Every lane takes part; each step moves to a lower index.
__device__ __forceinline__ void ancestor_words(int node, int par_lo, int par_hi, int32_t* dev_status,
                                               uint64_t& w0, uint64_t& w1) {
  int a = node;
  w0 = w1 = 0ull;
  for (int step = 0; step < 128; ++step) {
    if (!__any(a >= 0)) break;
    const uint64_t bit = 1ull << (a & 63);
    w0 |= (a >= 0 && a < 64) ? bit : 0ull;
    w1 |= (a >= 64) ? bit : 0ull;
    const int plo = __shfl(par_lo, a & 63, PTD_WAVE);
    const int phi = __shfl(par_hi, a & 63, PTD_WAVE);
    int nx = a >= 64 ? phi : plo;
    if (a < 0) {
      nx = -1;
    } else if (nx < -1 || nx >= a) {  // not topological
      ptd::report(dev_status, PTD_ERR_BAD_TREE);
      nx = -1;
    }
    a = nx;
  }
}

template <int D>
__global__ void __launch_bounds__(kF32Threads, 2) k_attn_f32(AttnParams p) {
  constexpr int KJ = D / 16;  // 16-byte loads of a K or Q fragment
  constexpr int H = D / 64;   // 64-column halves of V and O
  __shared__ __attribute__((aligned(16))) float so[kF32Waves][kF32Rows][D];
  __shared__ float2 sml[kF32Waves][kF32Rows];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, l4 = lane >> 4;
  int id;
  // (a grid of three dimensions: one of them holds fewer than 2^32 threads)
  const int bid = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
  logical_block(bid, p.B * p.Hkv * p.passes * p.splits, p.B * p.Hkv, false, id);
  const int split = id % p.splits;
  int rest = id / p.splits;
  const int r0 = (rest % p.passes) * kF32Rows;
  rest /= p.passes;
  const int g = rest % p.Hkv, b = rest / p.Hkv;
  const int n_kv = p.kv_len[b];
  const int tl = live_nodes(p, b);
  if (n_kv < 0 || n_kv > p.L_cap - tl) {  // (no overflow near the int range)
    if (tid == 0) ptd::report(p.dev_status, PTD_ERR_KV_LEN);
    return;
  }
  const int N = n_kv + tl;
  const int csz = chunk_size(N, p.splits);
  const int start = split * csz, end = min(N, start + csz);
  if (p.splits > 1 && start >= end) return;  // empty split: the combine skips it

  // this lane's query row (padding nodes read row 0; their output is zero)
  const int r = min(r0 + l16, p.M - 1);
  const int node = r / p.G < tl ? r / p.G : 0;
  const bool live = r / p.G < tl;
  const float* qr = static_cast<const float*>(p.q) +
                    ((static_cast<size_t>(b) * p.T + node) * p.Hq + g * p.G + r % p.G) * D + 4 * l4;
  const size_t kvoff = (static_cast<size_t>(b) * p.Hkv + g) * p.L_cap * D;
  const float* kb = static_cast<const float*>(p.k) + kvoff + 4 * l4;
  const float* vb = static_cast<const float*>(p.v) + kvoff + 4 * l16;

  const int ntiles = end > start ? (end - start + kF32Keys - 1) / kF32Keys : 0;
  f32x4 qf[KJ], kf[KJ];
  auto load_k = [&](int t) __attribute__((always_inline)) {
    const float* src = kb + static_cast<size_t>(min(start + t * kF32Keys + l16, N - 1)) * D;
#pragma unroll
    for (int j = 0; j < KJ; ++j) kf[j] = *reinterpret_cast<const f32x4*>(src + 16 * j);
  };
  if (wave < ntiles) {
    load_k(wave);
#pragma unroll
    for (int j = 0; j < KJ; ++j) qf[j] = *reinterpret_cast<const f32x4*>(qr + 16 * j);
  }
  // ancestors of this lane's node, where the wave meets tree keys and no mask
  // rows are given
  uint64_t w0 = 0, w1 = 0;
  if (!p.mask && end > n_kv) {
    const int32_t* pb = p.parent + static_cast<size_t>(b) * p.T;
    const int lo = lane < tl ? pb[lane] : -1, hi = lane + 64 < tl ? pb[lane + 64] : -1;
    ancestor_words(live ? node : -1, lo, hi, p.dev_status, w0, w1);
  }

  f32x4 o[H][4];
#pragma unroll
  for (int h = 0; h < H; ++h)
#pragma unroll
    for (int f = 0; f < 4; ++f) o[h][f] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = kNegBig, l = 0.f;  // l: this lane's keys only
  for (int t = wave; t < ntiles; t += kF32Waves) {
    const int key0 = start + t * kF32Keys + 4 * l4;
    f32x4 vf[4][H];
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int h = 0; h < H; ++h)
        vf[e][h] = *reinterpret_cast<const f32x4*>(vb + static_cast<size_t>(min(key0 + e, N - 1)) * D + 64 * h);
    f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < KJ; ++j)
#pragma unroll
      for (int e = 0; e < 4; e += 2) {
        s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[j][e], qf[j][e], s0, 0, 0, 0);
        s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[j][e + 1], qf[j][e + 1], s1, 0, 0, 0);
      }
    if (t + kF32Waves < ntiles) load_k(t + kF32Waves);
    f32x4 s = (s0 + s1) * p.scale;
    if (start + (t + 1) * kF32Keys > min(n_kv, end)) {  // uniform: tree keys, or past the split
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int key = key0 + e;
        const int a = min(max(key - n_kv, 0), p.T - 1);
        const uint64_t word = p.mask ? p.mask[(static_cast<size_t>(b) * p.T + node) * p.W + (a >> 6)]
                                     : (a >= 64 ? w1 : w0);
        const bool vis = key < end && (key < n_kv || ((word >> (a & 63)) & 1ull) != 0);
        s[e] = vis ? s[e] : -INFINITY;
      }
    }
    float mx = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
    mx = fmaxf(m, max_xor32(max_xor16(mx)));
    const float alpha = expf(m - mx);
    m = mx;
    f32x4 pr;
#pragma unroll
    for (int e = 0; e < 4; ++e) pr[e] = expf(s[e] - mx);
    l = l * alpha + ((pr[0] + pr[1]) + (pr[2] + pr[3]));
#pragma unroll
    for (int h = 0; h < H; ++h)
#pragma unroll
      for (int f = 0; f < 4; ++f) o[h][f] *= alpha;
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int h = 0; h < H; ++h)
#pragma unroll
        for (int f = 0; f < 4; ++f)
          o[h][f] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[e][h][f], pr[e], o[h][f], 0, 0, 0);
  }

  // merge of the waves: lane (l16, l4) holds query l16, columns
  // 64 h + 16 l4 + 4 x + f of O in o[h][f][x]
  l = sum_xor32(sum_xor16(l));
  if (l4 == 0) sml[wave][l16] = make_float2(m, l);
  if (wave < ntiles) {
#pragma unroll
    for (int h = 0; h < H; ++h)
#pragma unroll
      for (int x = 0; x < 4; ++x)
        *reinterpret_cast<f32x4*>(&so[wave][l16][64 * h + 16 * l4 + 4 * x]) =
            f32x4{o[h][0][x], o[h][1][x], o[h][2][x], o[h][3][x]};
  }
  __syncthreads();
  const int nw = min(ntiles, kF32Waves);
  for (int x = tid; x < kF32Rows * D / 4; x += kF32Threads) {
    const int row = x / (D / 4), d = (x % (D / 4)) * 4;
    const int rr = r0 + row;
    if (rr >= p.M) break;
    float mm = kNegBig;
    for (int w = 0; w < nw; ++w) mm = fmaxf(mm, sml[w][row].x);
    float den = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int w = 0; w < nw; ++w) {
      const float2 ml = sml[w][row];
      const float f = expf(ml.x - mm);
      den = fmaf(f, ml.y, den);
      acc += *reinterpret_cast<const f32x4*>(&so[w][row][d]) * f;
    }
    if (p.splits > 1) {
      const size_t prow = ((static_cast<size_t>(split) * p.B + b) * p.Hkv + g) * p.M + rr;
      *reinterpret_cast<f32x4*>(p.part_o + prow * D + d) = acc;
      if (d == 0) p.part_ml[prow] = make_float2(mm, den);
      continue;
    }
    const int i = rr / p.G, hg = rr % p.G;
    const size_t off = ((static_cast<size_t>(b) * p.T + i) * p.Hq + g * p.G + hg) * D + d;
    f32x4 v = {0.f, 0.f, 0.f, 0.f};  // padding nodes: zero
    if (i < tl)
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = acc[e] / den;
    if (p.out_bf16) {
      const u32x2 w = {ptd::cvt_pk_bf16(v[0], v[1]), ptd::cvt_pk_bf16(v[2], v[3])};
      *reinterpret_cast<u32x2*>(static_cast<uint16_t*>(p.out) + off) = w;
    } else {
      *reinterpret_cast<f32x4*>(static_cast<float*>(p.out) + off) = v;
    }
  }
}

// ===========================================================================
// host planning
// ===========================================================================
struct Plan {
  bool mfma;
  int QB, WR, passes, rows_per_pass;
  int splits;  // KV splits, the largest a call may take: sizes the partials
  int splits_full, splits_live;  // of a call without and with tree_len
  float precise_full, precise_live;
  int nt;  // threads per k_attn_mfma workgroup (512, or 256 with two workgroups per CU)
  bool needs_mask;  // workspace has room for mask rows (fp32 inputs, trees over 128 nodes)
  // workspace: [partials][mask rows], each 256-byte aligned
  size_t partial_bytes, mask_bytes, total_bytes;
};

size_t align256(size_t n) { return (n + 255) & ~static_cast<size_t>(255); }

constexpr int kTargetBlocks = 256;  // one resident workgroup per CU on MI355X

bool make_plan(const ptd_attn_shape* s, int T, Plan* pl) {
  if (!s || s->B < 1 || s->Hq < 1 || s->Hkv < 1 || s->Hq % s->Hkv) return false;
  if (s->D != 64 && s->D != 128) return false;
  if (T < 1 || T > PTD_MAX_T || s->L_cap < 1) return false;  // (L_cap >= T: per entry point)
  if ((s->in_dtype != PTD_F32 && s->in_dtype != PTD_BF16) ||
      (s->out_dtype != PTD_F32 && s->out_dtype != PTD_BF16))
    return false;
  const long long M = static_cast<long long>(T) * (s->Hq / s->Hkv);
  if (M > (1 << 24)) return false;
  pl->mfma = s->in_dtype == PTD_BF16;
  if (pl->mfma) {
    const int mp = static_cast<int>(M < 256 ? M : 256);
    const int nblk = (mp + 15) / 16;
    // 8 waves: WR row groups of 16*QB rows (QB <= 2) x (8/WR) key groups.
    // Up to 64 rows: passes of 32 rows (QB = 1), so that the workgroups of a
    // (b, g) split its keys half as many ways: half the split partials for
    // the combine, with each key read by two passes sharing one L2
    // (measured on 32 heads x 64 rows x 2112 keys: 14.3 + 4.7 us against
    // 16.3 + 4.7 us for one 64-row pass and twice the splits).
    if (nblk <= 4) { pl->WR = 2; pl->QB = 1; }
    // 65-128 rows: passes of 64 (WR = 2, QB = 2), fewer waves reading each
    // sub-tile than one 128-row pass (measured on 40 KV heads x 96 rows x
    // 4192 keys: 33.3 against 35.2 us).
    else if (nblk <= 8) { pl->WR = 2; pl->QB = 2; }
    // More than 128 rows: passes of 128 (WR = 4, QB = 2) rather than one
    // pass of up to 256 rows over eight row groups.  Every row-group wave
    // reads each K/V sub-tile from LDS, so four waves halve the LDS reads per
    // key; the passes share the keys through one XCD's L2 (measured on 8
    // KV heads x 256 rows x 32832 keys: 64.1 against 69.4 us).
    else { pl->WR = 4; pl->QB = 2; }
    // A batch of sequences in 128-row passes runs 256-thread workgroups (the
    // four row groups, one key group, a five-sub-tile ring in half of LDS),
    // two resident per CU: one's prologue and tail overlap the other's rounds
    // instead of following them, and their rounds drift apart instead of
    // meeting at one barrier (measured on ragged-16: 136.5 against 146.2 us
    // with three KV splits per sequence, 141.2 with two; a single sequence
    // was not faster: 68.1 against 67.3 us on 8 KV heads x 32832 keys).
    pl->nt = (pl->WR == 4 && s->B > 1) ? 256 : kThreads;
    pl->rows_per_pass = 16 * pl->QB * pl->WR;
    pl->passes = static_cast<int>((M + pl->rows_per_pass - 1) / pl->rows_per_pass);
    const long long items = static_cast<long long>(s->B) * s->Hkv * pl->passes;
    const auto splits_for = [&](int target) {
      int sp = static_cast<int>(target / items);
      const int max_by_len = (s->L_cap + 255) / 256;  // at least ~256 keys per split
      if (sp > max_by_len) sp = max_by_len;
      if (sp < 1) sp = 1;
      return sp > 64 ? 64 : sp;
    };
    // Several sequences may differ in length (kv_len is not known here):
    // twice the workgroups, so the dispatcher can even out long and short
    // ones (measured on 16 sequences of 512-8192 keys: 151-158 against
    // 167-171 us; a single sequence was slower with it).
    const int target = pl->nt == 256 ? 3 * kTargetBlocks : s->B > 1 ? 2 * kTargetBlocks : kTargetBlocks;
    pl->splits = pl->splits_full = pl->splits_live = splits_for(target);
    pl->precise_full = pl->precise_live = kPreciseFrac;
    if (pl->nt == 256) {
      // 256-thread workgroups, two per CU.  Exactly two per CU (512, `even` splits)
      // spare the third round of half the CUs, but lengths differ: where one
      // sequence is longer than the others its own chunks set the time, and more
      // splits are faster (16 x 40 nodes, 4 KV heads, one of 6104 keys and 15 of 64,
      // four / two splits: 54 / 83 us; all equal 108 / 115).  So only where the chunks
      // are short or a sequence fills the CUs alone, us with / without:
      //  - chunks of up to 512 keys without padding: over 613 drawn batches 0.87 of the
      //    time (at worst 1.07), one long among ones of 1/2 to 1/16 0.93 (1.21), among
      //    ones of 64 keys 1.00 (1.25); chunks of up to 640 keys 1.08 there (1.33);
      //  - of up to 288 keys with it, if they fill the 512 places (0.97, 0.99, 1.01): 16
      //    x 64 nodes x 480 keys 37.4 / 47.0, one long and 15 of 64 keys 32.6 / 35.3;
      //  - one split, which needs no combine: 24 x 36 x 508 keys 0.75-0.81 of the time
      //    of two; up to 704 keys without padding;
      //  - two sequences, each of which has a workgroup for 7/8 of the CUs alone,
      //    without padding (2 x 256 nodes x 832 keys 42.9 / 49.4, x 8000 99.7 / 112.9,
      //    2 x 211 nodes of 585-1171 keys 33.0 / 41.5; one of 64 keys 0.88-1.05 of the
      //    time), chunks of up to 1024 keys where the splits are more than 1.5 times
      //    fewer (0.86 of the time on average, one of 64 keys 0.95, at worst 1.10; from
      //    there on up to 1.12).
      // Longer splits carry fewer of a row's keys as hi + lo; half the threshold keeps
      // the error no larger (over drawn batches 0.975 of it on average, 1.009 at most).
      const int even = splits_for(2 * kTargetBlocks);
      const long long keys = (s->L_cap + even - 1LL) / even;
      const bool one_split = even == 1 && keys <= 544 && items >= 384;
      const bool one_short = even == 1 && keys <= 704;
      const bool few_keys = even > 1 && keys <= 288 && items * even >= 480;
      const bool few_short = even > 1 && keys <= 512 && items * even >= 400;
      const bool fills_alone = static_cast<long long>(s->Hkv) * pl->passes * even >= kTargetBlocks * 7 / 8 &&
                               keys <= (2 * pl->splits <= 3 * even ? 3072 : 1024);
      if (even < pl->splits && (one_split || one_short || few_keys || few_short || fills_alone)) {
        pl->splits_full = even;
        pl->precise_full = kPreciseFrac / 2;
        if (one_split || few_keys) {
          pl->splits_live = even;
          pl->precise_live = kPreciseFrac / 2;
        }
      }
    }
  } else {
    // fp32: 16-row workgroups; the keys are split while workgroups are fewer
    // than CUs and a split keeps at least 512 keys x 64 columns (about 4 us of
    // matrix work; the combine of the splits costs about as much)
    pl->WR = pl->QB = 0;
    pl->nt = kF32Threads;
    pl->rows_per_pass = kF32Rows;
    pl->passes = static_cast<int>((M + kF32Rows - 1) / kF32Rows);
    const long long items = static_cast<long long>(s->B) * s->Hkv * pl->passes;
    const int max_by_len = static_cast<int>((static_cast<long long>(s->L_cap) * (s->D / 64) + 511) / 512);
    pl->splits = static_cast<int>(std::min<long long>(std::max<long long>(kTargetBlocks / items, 1), std::min(max_by_len, 64)));
    pl->splits_full = pl->splits_live = pl->splits;
    pl->precise_full = pl->precise_live = kPreciseFrac;
  }
  if (static_cast<long long>(s->B) * s->Hkv * pl->passes * pl->splits > 0x7FFFFFFFLL) return false;
  // the combine's grid: one workgroup per 8 (D = 128) or 16 (D = 64) rows of a (b, g)
  if (pl->splits > 1 && static_cast<long long>(s->B) * s->Hkv * ((M + 7) / 8) > 0x7FFFFFFFLL) return false;
  pl->needs_mask = !pl->mfma || T > 128;  // (fp32, T <= 128: room only, no mask pass)
  pl->partial_bytes = pl->splits > 1
      ? align256(static_cast<size_t>(pl->splits) * s->B * s->Hkv * M * (s->D + 2) * sizeof(float))
      : 0;
  pl->mask_bytes = align256(static_cast<size_t>(s->B) * T * ((T + 63) / 64) * sizeof(uint64_t));
  pl->total_bytes = pl->partial_bytes + (pl->needs_mask ? pl->mask_bytes : 0);
  return true;
}

template <int D, bool F8, bool PAGED>
void launch_mfma(const Plan& pl, const AttnParams& prm, hipStream_t st) {
  const dim3 grid(prm.B * prm.Hkv * pl.passes * pl.splits);
  if (pl.nt == 256) {
    hipLaunchKernelGGL((k_attn_mfma<D, 2, 4, F8, PAGED, 256>), grid, dim3(256), 0, st, prm);
    return;
  }
  const dim3 block(kThreads);
#define PTD_MFMA_CASE(qb_, wr_) \
  if (pl.QB == qb_ && pl.WR == wr_) { hipLaunchKernelGGL((k_attn_mfma<D, qb_, wr_, F8, PAGED>), grid, block, 0, st, prm); return; }
  PTD_MFMA_CASE(1, 2) PTD_MFMA_CASE(2, 2) PTD_MFMA_CASE(2, 4)
#undef PTD_MFMA_CASE
}

}  // namespace

extern "C" size_t ptd_tree_attention_workspace_bytes(const ptd_attn_shape* shape, int32_t T) {
  Plan pl;
  if (!make_plan(shape, T, &pl)) return 0;
  return pl.total_bytes;
}

// ---------------------------------------------------------------------------
// Allocation-free variant: the scratch is a fixed device array.  In host code
// `scratch` names a host-side stand-in, never the device memory: its device
// address is looked up once per GPU (hipGetSymbolAddress with that GPU
// current) and only that address is handed to kernels.
// ---------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[PTD_NOALLOC_SCRATCH_BYTES];

namespace {

constexpr int kMaxScratchDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxScratchDevices] = {};

// Device address of the current GPU's scratch array (null on failure).
void* scratch_device_ptr() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxScratchDevices) return nullptr;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) {
      (void)hipGetLastError();  // clear the sticky error of the failed lookup
      return nullptr;
    }
    g_scratch_ptr[dev] = ptr;
  }
  return g_scratch_ptr[dev];
}

}  // namespace

namespace {

// The attention call on contiguous caches (page_table null) or paged ones.
int attention_impl(const void* q, const void* k_cache, const void* v_cache,
                   const int32_t* kv_len, const int32_t* tree_len, const int32_t* parent,
                   int32_t T, void* out,
                   const ptd_attn_shape* shape, const uint64_t* mask, void* workspace,
                   size_t workspace_bytes, int32_t* dev_status, void* stream,
                   const int32_t* page_table, int page_shift, int max_pages, int num_pages,
                   bool f8 = false, const float* k_scale = nullptr,
                   const float* v_scale = nullptr, bool noalloc = false) {
  PTD_RETURN_IF(!q || !k_cache || !v_cache || !kv_len || !parent || !out || !shape,
                PTD_ERR_NULL);
  if (shape->in_dtype != PTD_F32 && shape->in_dtype != PTD_BF16) return PTD_ERR_DTYPE;
  if (shape->out_dtype != PTD_F32 && shape->out_dtype != PTD_BF16) return PTD_ERR_DTYPE;
  Plan pl;
  PTD_RETURN_IF(!make_plan(shape, T, &pl), PTD_ERR_SHAPE);
  // every tree row must fit unless tree sizes come with the call
  PTD_RETURN_IF(!tree_len && shape->L_cap < T, PTD_ERR_SHAPE);
  PTD_RETURN_IF(!ptd_aligned(q, 16) || !ptd_aligned(k_cache, 16) || !ptd_aligned(v_cache, 16) ||
                    !ptd_aligned(out, 16) || (mask && !ptd_aligned(mask, 8)),
                PTD_ERR_ALIGN);
  if (!pl.mfma) PTD_RETURN_IF(shape->Hkv > 65535 || shape->B > 65535, PTD_ERR_SHAPE);
  const size_t mask_need = pl.needs_mask && !mask ? pl.mask_bytes : 0;
  // fp32 inputs: the split is an option, taken where its partials fit the scratch
  // (a workspace that is not aligned for them counts as none)
  const size_t room = noalloc ? PTD_NOALLOC_SCRATCH_BYTES
                              : workspace && ptd_aligned(workspace, 256) ? workspace_bytes : 0;
  if (!pl.mfma && pl.splits > 1 && pl.partial_bytes + mask_need > room) {
    pl.splits_full = pl.splits_live = 1;
    pl.partial_bytes = 0;
  }
  // (the workspace holds the larger count's partials either way)
  pl.splits = tree_len ? pl.splits_live : pl.splits_full;
  const bool build_mask = mask_need > 0 && T > 128;
  const size_t need = pl.partial_bytes + mask_need;
  if (noalloc && need > 0) {  // the fixed scratch array stands in for the workspace
    PTD_RETURN_IF(need > PTD_NOALLOC_SCRATCH_BYTES, PTD_ERR_SCRATCH);
    workspace = scratch_device_ptr();
    PTD_RETURN_IF(!workspace, PTD_ERR_HIP);
    workspace_bytes = PTD_NOALLOC_SCRATCH_BYTES;
  }
  if (need > 0) {
    PTD_RETURN_IF(!workspace, PTD_ERR_WORKSPACE);
    PTD_RETURN_IF(workspace_bytes < need, PTD_ERR_WORKSPACE);
    PTD_RETURN_IF(!ptd_aligned(workspace, 256), PTD_ERR_ALIGN);
  }
  hipStream_t st = static_cast<hipStream_t>(stream);
  unsigned char* ws = static_cast<unsigned char*>(workspace);
  if (build_mask) {
    uint64_t* mws = reinterpret_cast<uint64_t*>(ws + pl.partial_bytes);
    const int rc = ptd_launch_tree_mask(parent, tree_len, shape->B, T, mws, nullptr, dev_status, st);
    if (rc != PTD_OK) return rc;
    mask = mws;
  }
  AttnParams prm;
  prm.q = q;
  prm.k = k_cache;
  prm.v = v_cache;
  prm.kv_len = kv_len;
  prm.parent = parent;
  prm.tree_len = tree_len;
  prm.k_scale = k_scale;
  prm.v_scale = v_scale;
  prm.mask = pl.needs_mask ? mask : nullptr;  // (fp32, T <= 128: used when given)
  prm.out = out;
  prm.part_o = pl.splits > 1 ? reinterpret_cast<float*>(ws) : nullptr;
  prm.part_ml = nullptr;
  prm.dev_status = dev_status;
  prm.B = shape->B;
  prm.T = T;
  prm.Hq = shape->Hq;
  prm.Hkv = shape->Hkv;
  prm.G = shape->Hq / shape->Hkv;
  prm.M = T * prm.G;
  prm.L_cap = shape->L_cap;
  prm.W = (T + 63) / 64;
  prm.splits = pl.splits;
  prm.passes = pl.passes;
  prm.rows_per_pass = pl.rows_per_pass;
  prm.scale = shape->scale > 0.f ? shape->scale : 1.0f / sqrtf(static_cast<float>(shape->D));
  prm.c = prm.scale * kLog2e;
  prm.precise = tree_len ? pl.precise_live : pl.precise_full;
  prm.out_bf16 = shape->out_dtype == PTD_BF16;
  prm.page_table = page_table;
  prm.page_shift = page_shift;
  prm.max_pages = max_pages;
  prm.num_pages = num_pages;
  if (pl.splits > 1) {
    const size_t rows = static_cast<size_t>(pl.splits) * prm.B * prm.Hkv * prm.M;
    prm.part_ml = reinterpret_cast<float2*>(prm.part_o + rows * shape->D);
  }
  if (pl.mfma) {
    const auto launch = [&](auto paged) {
      constexpr bool kPaged = decltype(paged)::value;
      if (f8) launch_mfma<128, true, kPaged>(pl, prm, st);  // (D = 128 checked by the entry point)
      else if (shape->D == 128) launch_mfma<128, false, kPaged>(pl, prm, st);
      else launch_mfma<64, false, kPaged>(pl, prm, st);
    };
    if (page_table) launch(std::true_type{});
    else launch(std::false_type{});
  } else {
    const dim3 grid(pl.passes * pl.splits, prm.Hkv, prm.B);
    if (shape->D == 128) hipLaunchKernelGGL(k_attn_f32<128>, grid, dim3(kF32Threads), 0, st, prm);
    else hipLaunchKernelGGL(k_attn_f32<64>, grid, dim3(kF32Threads), 0, st, prm);
  }
  if (pl.splits > 1) {
    const int rpb = 256 / (shape->D / 4);  // rows per combine workgroup
    const dim3 grid(static_cast<unsigned>(static_cast<long long>(prm.B) * prm.Hkv *
                                          ((prm.M + rpb - 1) / rpb)));
    // U = splits loaded at once: the fewest of 2, 4, 8, 16 covering them
    // (16 splits in one group of loads rather than two: 72.4 against 76.4
    // us per call on 8 KV heads x 256 rows x 32832 keys)
    const int u = pl.splits <= 2 ? 2 : pl.splits <= 4 ? 4 : pl.splits <= 8 ? 8 : 16;
#define PTD_COMBINE(d_, u_)                                                                      \
  if (shape->D == d_ && u == u_) {                                                               \
    if (pl.mfma) hipLaunchKernelGGL((k_attn_combine<d_, u_, false>), grid, dim3(256), 0, st, prm); \
    else hipLaunchKernelGGL((k_attn_combine<d_, u_, true>), grid, dim3(256), 0, st, prm);        \
  }
    PTD_COMBINE(128, 2) PTD_COMBINE(128, 4) PTD_COMBINE(128, 8) PTD_COMBINE(128, 16)
    PTD_COMBINE(64, 2) PTD_COMBINE(64, 4) PTD_COMBINE(64, 8) PTD_COMBINE(64, 16)
#undef PTD_COMBINE
  }
  return ptd_launch_status();
}

}  // namespace

extern "C" int ptd_tree_attention(const void* q, const void* k_cache, const void* v_cache,
                                  const int32_t* kv_len, const int32_t* parent, int32_t T,
                                  void* out, const ptd_attn_shape* shape,
                                  const uint64_t* mask, void* workspace,
                                  size_t workspace_bytes, int32_t* dev_status,
                                  void* stream) {
  return attention_impl(q, k_cache, v_cache, kv_len, nullptr, parent, T, out, shape, mask,
                        workspace, workspace_bytes, dev_status, stream, nullptr, 0, 0, 0);
}

extern "C" int ptd_tree_attention_ragged(const void* q, const void* k_cache, const void* v_cache,
                                         const int32_t* kv_len, const int32_t* tree_len,
                                         const int32_t* parent, int32_t T, void* out,
                                         const ptd_attn_shape* shape, const uint64_t* mask,
                                         void* workspace, size_t workspace_bytes,
                                         int32_t* dev_status, void* stream) {
  return attention_impl(q, k_cache, v_cache, kv_len, tree_len, parent, T, out, shape, mask,
                        workspace, workspace_bytes, dev_status, stream, nullptr, 0, 0, 0);
}

extern "C" int ptd_tree_attention_noalloc(const void* q, const void* k_cache, const void* v_cache,
                                          const int32_t* kv_len, const int32_t* tree_len,
                                          const int32_t* parent, int32_t T, void* out,
                                          const ptd_attn_shape* shape, const uint64_t* mask,
                                          int32_t* dev_status, void* stream) {
  return attention_impl(q, k_cache, v_cache, kv_len, tree_len, parent, T, out, shape, mask,
                        nullptr, 0, dev_status, stream, nullptr, 0, 0, 0, false, nullptr, nullptr,
                        true);
}

extern "C" int ptd_tree_attention_fp8kv(const void* q, const void* k_cache, const void* v_cache,
                                        const float* k_scale, const float* v_scale,
                                        const int32_t* kv_len, const int32_t* tree_len,
                                        const int32_t* parent, int32_t T, void* out,
                                        const ptd_attn_shape* shape, void* workspace,
                                        size_t workspace_bytes, int32_t* dev_status,
                                        void* stream) {
  PTD_RETURN_IF(!shape, PTD_ERR_NULL);
  PTD_RETURN_IF(shape->in_dtype != PTD_BF16, PTD_ERR_DTYPE);  // bf16 queries (the MFMA path)
  PTD_RETURN_IF(shape->D != 128, PTD_ERR_SHAPE);
  PTD_RETURN_IF((k_scale && !ptd_aligned(k_scale, 4)) || (v_scale && !ptd_aligned(v_scale, 4)),
                PTD_ERR_ALIGN);
  return attention_impl(q, k_cache, v_cache, kv_len, tree_len, parent, T, out, shape, nullptr,
                        workspace, workspace_bytes, dev_status, stream, nullptr, 0, 0, 0, true,
                        k_scale, v_scale);
}

namespace {

// Checks of a page description; the page-size shift on success.
int paged_args(const ptd_kv_pages* kv, const ptd_attn_shape* shape, int* shift) {
  PTD_RETURN_IF(!kv || !shape, PTD_ERR_NULL);
  PTD_RETURN_IF(!kv->k_pages || !kv->v_pages || !kv->page_table, PTD_ERR_NULL);
  PTD_RETURN_IF(shape->in_dtype != PTD_BF16, PTD_ERR_DTYPE);  // the MFMA path only
  const int ps = kv->page_size;
  PTD_RETURN_IF(ps < 32 || ps > (1 << 20) || (ps & (ps - 1)) != 0, PTD_ERR_SHAPE);
  PTD_RETURN_IF(kv->max_pages < 1 || kv->num_pages < 1, PTD_ERR_SHAPE);
  PTD_RETURN_IF(static_cast<long long>(kv->max_pages) * ps != shape->L_cap, PTD_ERR_SHAPE);
  int sh = 0;
  while ((1 << sh) < ps) ++sh;
  *shift = sh;
  return PTD_OK;
}

}  // namespace

extern "C" int ptd_tree_attention_paged(const void* q, const ptd_kv_pages* kv,
                                        const int32_t* kv_len, const int32_t* tree_len,
                                        const int32_t* parent, int32_t T,
                                        void* out, const ptd_attn_shape* shape,
                                        const uint64_t* mask, void* workspace,
                                        size_t workspace_bytes, int32_t* dev_status,
                                        void* stream) {
  int shift = 0;
  const int rc = paged_args(kv, shape, &shift);
  if (rc != PTD_OK) return rc;
  return attention_impl(q, kv->k_pages, kv->v_pages, kv_len, tree_len, parent, T, out, shape, mask,
                        workspace, workspace_bytes, dev_status, stream, kv->page_table, shift,
                        kv->max_pages, kv->num_pages);
}

extern "C" int ptd_tree_attention_paged_fp8kv(const void* q, const ptd_kv_pages* kv,
                                              const float* k_scale, const float* v_scale,
                                              const int32_t* kv_len, const int32_t* tree_len,
                                              const int32_t* parent, int32_t T, void* out,
                                              const ptd_attn_shape* shape, void* workspace,
                                              size_t workspace_bytes, int32_t* dev_status,
                                              void* stream) {
  int shift = 0;
  const int rc = paged_args(kv, shape, &shift);
  if (rc != PTD_OK) return rc;
  PTD_RETURN_IF(shape->D != 128, PTD_ERR_SHAPE);
  PTD_RETURN_IF((k_scale && !ptd_aligned(k_scale, 4)) || (v_scale && !ptd_aligned(v_scale, 4)),
                PTD_ERR_ALIGN);
  return attention_impl(q, kv->k_pages, kv->v_pages, kv_len, tree_len, parent, T, out, shape,
                        nullptr, workspace, workspace_bytes, dev_status, stream, kv->page_table,
                        shift, kv->max_pages, kv->num_pages, true, k_scale, v_scale);
}
