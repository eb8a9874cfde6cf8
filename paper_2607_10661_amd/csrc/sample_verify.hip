// Sampling verification of a draft tree (Sec. 3.2 "sampling decoding
// strategy"; App. E recursive candidate-tree sampling; App. F proof of
// distributional consistency).
//
// P_v = softmax(logits row of v / temperature); row 0 is the last committed
// token n_0 (the parent of every root), row v + 1 is node v.  From n_0 the
// children of the current node are examined in index order; child n (token
// t_n) is accepted iff u_node[n] < P_v[t_n] / S, S being the mass of P_v not
// yet rejected at this node (App. F divides by it).  A rejected token's
// probability becomes 0, so a later sibling with the same token is rejected.
// On acceptance the walk moves to n; when every child is rejected the node is
// the terminal and the bonus token is drawn by inverse CDF (index order) from
// the residual distribution with u_bonus[row].
//
// Kernels
//   k_block_stats    one wave per (block of 2048 vocabulary entries, logits
//                    row), four per workgroup (k_block_stats_wg: one
//                    workgroup per block, for calls with few blocks): the
//                    largest logit m_b and z_b = sum 2^(l c - k_b) over the
//                    block, c = log2(e) / temperature and k_b the integer
//                    nearest to m_b c; each term an fp32 exponential with its
//                    argument's rounding compensated (~1.2e-7 relative), added
//                    in fp64.
//   k_verify_sample  one workgroup of 1024 threads per sequence.  Each row's
//                    k = max_b k_b and normalizer z = sum_b z_b 2^(k_b - k)
//                    (exact scalings) are formed in LDS; the tree, the
//                    uniforms and every node's probability under its parent's
//                    row (numerator in fp64) are staged.  Each level of the walk lists the
//                    current node's children in index order with ballots, and
//                    one thread takes the accept / reject decisions in order;
//                    rejected tokens are marked in an LDS bitmap (one bit per
//                    vocabulary entry).  Bonus draw: the block sums of the
//                    terminal's row, less the rejected terms, locate the block
//                    where the running total passes u * W; that block's 2048
//                    terms are recomputed (the same arithmetic) and scanned by
//                    all threads.
#include <math.h>

#include "ptd_common.hpp"

namespace {

constexpr int kStatThreads = 256;
constexpr int kBlock = 2048;  // vocabulary entries per statistics block
constexpr int kWalkThreads = 1024;
constexpr int kWalkWaves = kWalkThreads / PTD_WAVE;
constexpr int kMaxVocab = 262144;  // LDS bitmap of rejected tokens: 32 KB
constexpr int kMaxBlocks = kMaxVocab / kBlock;
constexpr int kStagedStats = 4096;  // block statistics kept in LDS by the walk (64 KB)

template <bool BF16>
__device__ __forceinline__ float logit(const void* row, int y) {
  if constexpr (BF16) return ptd::bf16_to_f32(static_cast<const uint16_t*>(row)[y]);
  else return static_cast<const float*>(row)[y];
}

__device__ __forceinline__ double shfl_up_f64(double x, int d) {
  const uint64_t u = __double_as_longlong(x);
  const uint32_t lo = __shfl_up(static_cast<uint32_t>(u), d, PTD_WAVE);
  const uint32_t hi = __shfl_up(static_cast<uint32_t>(u >> 32), d, PTD_WAVE);
  return __longlong_as_double(static_cast<long long>((static_cast<uint64_t>(hi) << 32) | lo));
}
// One DPP step of a wave scan on an fp64 value (both halves moved with the
// same control; lanes outside the row or the row mask receive +0.0).
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_f64(double x) {
  const uint64_t u = __double_as_longlong(x);
  const uint32_t lo = static_cast<uint32_t>(
      __builtin_amdgcn_update_dpp(0, static_cast<int>(static_cast<uint32_t>(u)), CTRL, ROWS, 0xF, false));
  const uint32_t hi = static_cast<uint32_t>(
      __builtin_amdgcn_update_dpp(0, static_cast<int>(static_cast<uint32_t>(u >> 32)), CTRL, ROWS, 0xF, false));
  return __longlong_as_double(static_cast<long long>((static_cast<uint64_t>(hi) << 32) | lo));
}
// Inclusive prefix sum over the wave on the vector ALU: row_shr 1, 2, 4, 8
// within rows of 16 lanes, then row_bcast:15 (into rows 1 and 3) and
// row_bcast:31 (into rows 2 and 3).
__device__ __forceinline__ double wave_incl_scan_f64(double x) {
  x += dpp_f64<0x111, 0xF>(x);
  x += dpp_f64<0x112, 0xF>(x);
  x += dpp_f64<0x114, 0xF>(x);
  x += dpp_f64<0x118, 0xF>(x);
  x += dpp_f64<0x142, 0xA>(x);
  x += dpp_f64<0x143, 0xC>(x);
  return x;
}
// Maximum over the wave in lane 63, the same steps (lanes without a partner
// keep their own value).
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_max(float x) {
  const int v = __builtin_bit_cast(int, x);
  return fmaxf(x, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(v, v, CTRL, ROWS, 0xF, false)));
}
__device__ __forceinline__ float wave_max_uniform(float x) {
  x = dpp_max<0x111, 0xF>(x);
  x = dpp_max<0x112, 0xF>(x);
  x = dpp_max<0x114, 0xF>(x);
  x = dpp_max<0x118, 0xF>(x);
  x = dpp_max<0x142, 0xA>(x);
  x = dpp_max<0x143, 0xC>(x);
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), 63));
}
__device__ __forceinline__ double readlane_f64(double x, int lane) {
  const uint64_t u = __double_as_longlong(x);
  const uint32_t lo = __builtin_amdgcn_readlane(static_cast<uint32_t>(u), lane);
  const uint32_t hi = __builtin_amdgcn_readlane(static_cast<uint32_t>(u >> 32), lane);
  return __longlong_as_double(static_cast<long long>((static_cast<uint64_t>(hi) << 32) | lo));
}

// A block's largest logit (the type's lowest value at least) and its sum of
// 2^(l c - k), k = block_ref(m).
struct RowStat {
  float m, unused;
  double z;
};

// c = log2(e) / temperature as an fp64 value and as c_hi + c_lo in fp32; plain: c
// is far inside the fp32 range.  l_min and d_min: -2000 / c and -200 / c.
struct Scale {
  double c;
  float c_hi, c_lo, l_min, d_min;
  bool plain;
};

constexpr float kFastRange = 800.0f;
constexpr float kGrid = 3072.0f;  // 1.5 * 2^11: adding it rounds |y| < 1024 to multiples of 2^-12
constexpr float kLowest = -3.402823466e38f;
constexpr float kLn2 = 0.69314718f;
// Integer reference of a block from its largest logit: powers of two rescale
// sums between references exactly.
__device__ __forceinline__ double block_ref(float m, const Scale& sc) {
  return rint(static_cast<double>(m) * sc.c);
}
// How a block's terms are formed (uniform over the block).
__device__ __forceinline__ bool fast_ref(double k, const Scale& sc) { return sc.plain && fabs(k) <= kFastRange; }
// l c - k in fp64, the product rounded first: k is the rounded product's integer,
// and far from 0 the product's rounding error alone exceeds 1.
__device__ __forceinline__ double scaled(float l, double k, const Scale& sc) {
#pragma clang fp contract(off)
  const double lc = static_cast<double>(l) * sc.c;
  return lc - k;
}
// A term as p (1 + e ln 2): p = 2^x in fp32 with e the rest of the exponent, which
// enters to first order.  The maximum is the one that keeps a NaN.
//
// Fast: 2^(l c - k) for |k| <= kFastRange.  l c is rounded to a multiple of 2^-12
// by one FMA, so the subtractions of kGrid and of k are exact; the rest of l c is
// at most 2^-13, found by two FMAs (second order below 6e-9).  The term is within
// about one ulp of v_exp_f32 (~1.2e-7 relative) of the exact value; it is 0 far
// below the reference.  Where l c overflows (l = -inf, the type's lowest value)
// it is NaN without the bound l_min, at which the term has long been 0.
__device__ __forceinline__ void fast_parts(float l, float kf, const Scale& sc, float& p, float& e) {
  const float t = fmaf(l, sc.c_hi, kGrid);
  const float y = t - kGrid;
  e = fmaf(l, sc.c_lo, fmaf(l, sc.c_hi, -y));
  p = __builtin_amdgcn_exp2f(y - kf);
}
// Far: 2^((l - m) c) for any other reference (low temperatures, large logits), 0
// from the bound far_low on.  fp32 logits keep the rounding of l - m (TwoSum).  The
// difference of bf16 logits is exact unless one of them is 2^16 times the other;
// rounded, it changes a term 2^x by at most x 2^-25 ln 2, 1.1e-8 of the block's
// largest.
__device__ __forceinline__ float far_low(float m, const Scale& sc) {
  return m + fminf(sc.d_min, -fabsf(m) * 0x1p-22f);  // (below m, however large m is)
}
template <bool BF16>
__device__ __forceinline__ void far_parts(float l, float m, float low, const Scale& sc, float& p, float& e) {
  l = __builtin_elementwise_maximum(l, low);
  const float d = l - m;
  const float x = d * sc.c_hi;
  e = fmaf(d, sc.c_hi, -x);
  if constexpr (!BF16) {
    const float bb = d - l;
    e = fmaf((l - (d - bb)) + (-m - bb), sc.c_hi, e);
  }
  e = fmaf(d, sc.c_lo, e);
  p = __builtin_amdgcn_exp2f(x);
}
__device__ __forceinline__ float one_term(float p, float e) { return fmaf(p * e, kLn2, p); }
// Sum of two terms, the correction applied once; the same bits as one_term's where
// the other term is 0, so what is left of a block's sum without its only entry
// with mass is 0.  k_block_stats is bound by its vector instructions: 11 per
// entry with fast terms (an exponential counted as two), 12 with their bound,
// 11 (bf16) or 16 with far terms.  1040 rows x 128256 bf16, whole calls: 57 us;
// 64 where every block is far (temperature 0.02, logits of deviation 4; 176 with
// fp64 terms there, 69.5 with far terms of 19 instructions everywhere); 67.5
// with every third entry masked (202 with fp64 terms).
__device__ __forceinline__ float two_terms(float p0, float e0, float p1, float e1) {
  return fmaf(fmaf(p1, e1, p0 * e0), kLn2, p0 + p1);
}
// Blocks of the type's lowest values (masks): neighbouring values there are more
// than 1e10 temperatures apart.
constexpr float kMasked = -1.0e38f;
__device__ __forceinline__ float masked_term(float l, float m) { return l == m ? 1.0f : 0.0f; }
// Temperatures at the ends of the fp32 range.
__device__ __noinline__ float wide_term(float l, float m, double c) {
  return static_cast<float>(exp2((static_cast<double>(l) - static_cast<double>(m)) * c));
}
// A term of a block (m, k), and what it is a multiple of: term * scale is
// 2^(l c - k), for the sums of k_block_stats and for the bonus draw alike.
template <bool BF16>
__device__ __forceinline__ float block_term(float l, float m, double k, const Scale& sc) {
  float p, e;
  if (fast_ref(k, sc)) fast_parts(__builtin_elementwise_maximum(l, sc.l_min), static_cast<float>(k), sc, p, e);
  else if (!sc.plain) return wide_term(l, m, sc.c);
  else if (m < kMasked) return masked_term(l, m);
  else far_parts<BF16>(l, m, far_low(m, sc), sc, p, e);
  return one_term(p, e);
}
__device__ __forceinline__ double block_scale(float m, double k, const Scale& sc) {
  return fast_ref(k, sc) ? 1.0 : exp2(scaled(m, k, sc));
}
// 2^d for an integer d <= 0 (0 far below the fp64 range)
__device__ __forceinline__ double pow2i(double d) { return ldexp(1.0, static_cast<int>(fmax(d, -4000.0))); }

using u32x4 = uint32_t __attribute__((ext_vector_type(4)));

// the values of a 16-byte chunk of a row
template <bool BF16>
__device__ __forceinline__ void chunk_vals(const u32x4& c, float (&x)[BF16 ? 8 : 4]) {
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    if constexpr (BF16) {
      x[2 * w] = ptd::bf16_lo(c[w]);
      x[2 * w + 1] = ptd::bf16_hi(c[w]);
    } else {
      x[w] = __uint_as_float(c[w]);
    }
  }
}

// The whole 16-byte chunks of block [y0, y1) of a row that may start at any
// element address, and one edge element per lane: the elements before the
// block's first 16-byte boundary and after its last whole chunk (fewer than
// two chunks).
template <bool BF16>
struct BlockSpan {
  const u32x4* chunks;
  int nch;
  int edge;  // this lane's edge element, -1: none
  __device__ BlockSpan(const char* row, int y0, int y1, int lane) {
    constexpr int E = BF16 ? 8 : 4, ES = BF16 ? 2 : 4;
    const char* p = row + static_cast<size_t>(y0) * ES;
    const int head = min(y1 - y0, static_cast<int>((0u - static_cast<uint32_t>(reinterpret_cast<uintptr_t>(p))) & 15u) / ES);
    chunks = reinterpret_cast<const u32x4*>(p + head * ES);
    nch = (y1 - y0 - head) / E;
    const int y = lane < head ? y0 + lane : y0 + head + nch * E + (lane - head);
    edge = y < y1 ? y : -1;
  }
};

constexpr float kNone = -0x1.92p+99f;  // bf16 0xF149, about -1e30
__device__ __forceinline__ float max3(float a, float b, float c) {
  float r;  // (fmaxf of freshly loaded bits costs two more instructions to quiet NaNs)
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}
// Largest of a lane's chunks and its edge element.
template <bool BF16, int N>
__device__ __forceinline__ float chunks_max(const u32x4 (&raw)[N], float le) {
  constexpr int E = BF16 ? 8 : 4;
  float m = le;
#pragma unroll
  for (int j = 0; j < N; ++j) {
    float x[E];
    chunk_vals<BF16>(raw[j], x);
#pragma unroll
    for (int e = 0; e < E; e += 2) m = max3(x[e], x[e + 1], m);
  }
  return m;
}
// Sum of the terms of a lane's chunks J0 .. J1 - 1 by pairs, added to z.
template <bool BF16, int J0, int J1, int N, class Pair>
__device__ __forceinline__ double chunks_sum(const u32x4 (&raw)[N], double z, Pair pair) {
  constexpr int E = BF16 ? 8 : 4;
#pragma unroll
  for (int j = J0; j < J1; ++j) {
    float x[E];
    chunk_vals<BF16>(raw[j], x);
#pragma unroll
    for (int e = 0; e < E; e += 2)  // pairs added in fp32 (one rounding, 2^-24), then fp64
      z += static_cast<double>(pair(x[e], x[e + 1]));
  }
  return z;
}
// Sum of the terms of a lane's chunks and its edge element for any block: masked
// entries (-inf or overflowing) count 0.
template <bool BF16, int N>
__device__ __forceinline__ double chunks_sum_any(const u32x4 (&raw)[N], float le, float m, double k,
                                                 const Scale& sc) {
  const double z = static_cast<double>(block_term<BF16>(le, m, k, sc));
  if (fast_ref(k, sc)) {  // uniform
    const float kf = static_cast<float>(k);
    return chunks_sum<BF16, 0, N>(raw, z, [&](float a, float b) {
      float p0, e0, p1, e1;
      fast_parts(__builtin_elementwise_maximum(a, sc.l_min), kf, sc, p0, e0);
      fast_parts(__builtin_elementwise_maximum(b, sc.l_min), kf, sc, p1, e1);
      return two_terms(p0, e0, p1, e1);
    });
  }
  const double f = block_scale(m, k, sc);
  if (!sc.plain)
    return f * chunks_sum<BF16, 0, N>(raw, z, [&](float a, float b) {
      return wide_term(a, m, sc.c) + wide_term(b, m, sc.c);
    });
  if (m < kMasked)
    return f * chunks_sum<BF16, 0, N>(raw, z, [&](float a, float b) {
      return masked_term(a, m) + masked_term(b, m);
    });
  const float low = far_low(m, sc);
  return f * chunks_sum<BF16, 0, N>(raw, z, [&](float a, float b) {
    float p0, e0, p1, e1;
    far_parts<BF16>(a, m, low, sc, p0, e0);
    far_parts<BF16>(b, m, low, sc, p1, e1);
    return two_terms(p0, e0, p1, e1);
  });
}

// Block reference, then the block's sum of terms relative to it: one wave per
// (block, row), four blocks per workgroup, no workgroup barrier, cross-lane
// steps on the vector ALU.  Chunks of 16 bytes (4 per lane for bf16, 8 for
// fp32, lane-interleaved) are all issued before the first is used.  1040 rows x
// 128256 bf16: 50.4 us (5.3 TB/s, what a copy reaches) against 64.1 with the
// longer term, guarded chunks and reductions through LDS.
template <bool BF16>
__global__ void __launch_bounds__(kStatThreads)
k_block_stats(const void* __restrict__ logits, int V, long long ld, int nblk, Scale sc,
              RowStat* __restrict__ stats) {
  constexpr int E = BF16 ? 8 : 4;
  constexpr int CPL = kBlock / E / PTD_WAVE;  // chunks per lane: 4 (bf16) or 8 (fp32)
  const int lane = threadIdx.x & 63;
  const int blk = blockIdx.x * (kStatThreads / PTD_WAVE) + (threadIdx.x >> 6);
  const int r = blockIdx.y;
  if (blk >= nblk) return;  // whole wave
  const char* row = static_cast<const char*>(logits) + static_cast<size_t>(r) * ld * (BF16 ? 2 : 4);
  const int y0 = blk * kBlock, y1 = min(V, y0 + kBlock);
  const BlockSpan<BF16> sp(row, y0, y1, lane);
  // missing chunks and edges hold kNone: terms of 0
  const uint32_t none = BF16 ? 0xF149F149u : __float_as_uint(kNone);
  u32x4 raw[CPL];
  if (sp.nch == CPL * PTD_WAVE) {  // uniform: a whole block of an aligned row
#pragma unroll
    for (int j = 0; j < CPL; ++j) raw[j] = sp.chunks[j * PTD_WAVE + lane];
  } else {
#pragma unroll
    for (int j = 0; j < CPL; ++j) {
      const int c = j * PTD_WAVE + lane;
      raw[j] = u32x4{none, none, none, none};
      if (c < sp.nch) raw[j] = sp.chunks[c];
    }
  }
  const float le = sp.edge >= 0 ? logit<BF16>(row, sp.edge) : kNone;
  float m = wave_max_uniform(chunks_max<BF16>(raw, le));
  double k = block_ref(m, sc);
  double z = __builtin_nan("");
  if (m > kNone && fast_ref(k, sc)) {  // uniform
    const float kf = static_cast<float>(k);
    const auto pair = [&](float a, float b) {
      float p0, e0, p1, e1;
      fast_parts(a, kf, sc, p0, e0);
      fast_parts(b, kf, sc, p1, e1);
      return two_terms(p0, e0, p1, e1);
    };
    float p, e;
    fast_parts(le, kf, sc, p, e);
    z = chunks_sum<BF16, 0, 1>(raw, static_cast<double>(one_term(p, e)), pair);
    if (!__any(!(z == z))) z = chunks_sum<BF16, 1, CPL>(raw, z, pair);  // (masks are found early)
  }
  if (__any(!(z == z))) {  // uniform: far logits, or masks that overflow l c
    const uint32_t ninf = BF16 ? 0xFF80FF80u : 0xFF800000u;
#pragma unroll
    for (int j = 0; j < CPL; ++j)
      if (j * PTD_WAVE + lane >= sp.nch) raw[j] = u32x4{ninf, ninf, ninf, ninf};
    const float lx = sp.edge >= 0 ? le : -INFINITY;
    if (!(m > kNone)) {  // uniform: padding may have been taken for an entry
      m = fmaxf(wave_max_uniform(chunks_max<BF16>(raw, lx)), kLowest);
      k = block_ref(m, sc);
    }
    z = chunks_sum_any<BF16>(raw, lx, m, k, sc);
  }
  z = wave_incl_scan_f64(z);
  if (lane == PTD_WAVE - 1) stats[static_cast<size_t>(r) * nblk + blk] = RowStat{m, 0.0f, z};
}

// The same statistics with one workgroup per (block, row), one or two chunks
// per thread: the shorter latency per block where the blocks of a call are
// few (a single sequence's rows).
template <bool BF16>
__global__ void __launch_bounds__(kStatThreads)
k_block_stats_wg(const void* __restrict__ logits, int V, long long ld, int nblk, Scale sc,
                 RowStat* __restrict__ stats) {
  constexpr int E = BF16 ? 8 : 4;
  constexpr int NW = kStatThreads / PTD_WAVE;
  constexpr int CPT = kBlock / E / kStatThreads;  // chunks per thread: 1 (bf16) or 2
  __shared__ float s_max[NW];
  __shared__ double s_sum[NW];
  const int blk = blockIdx.x, r = blockIdx.y, tid = threadIdx.x, lane = tid & 63,
            wave = tid >> 6;
  const char* row = static_cast<const char*>(logits) + static_cast<size_t>(r) * ld * (BF16 ? 2 : 4);
  const int y0 = blk * kBlock, y1 = min(V, y0 + kBlock);
  const BlockSpan<BF16> sp(row, y0, y1, tid);
  const uint32_t ninf = BF16 ? 0xFF80FF80u : 0xFF800000u;
  u32x4 raw[CPT];
#pragma unroll
  for (int j = 0; j < CPT; ++j) {
    const int c = tid + j * kStatThreads;
    raw[j] = u32x4{ninf, ninf, ninf, ninf};
    if (c < sp.nch) raw[j] = sp.chunks[c];
  }
  const float le = sp.edge >= 0 ? logit<BF16>(row, sp.edge) : -INFINITY;
  float m = wave_max_uniform(chunks_max<BF16>(raw, le));
  if (lane == 0) s_max[wave] = m;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < NW; ++w) m = fmaxf(m, s_max[w]);
  m = fmaxf(m, kLowest);
  // (every entry by its own term: a wave of padding or masks costs no second pass)
  double z = wave_incl_scan_f64(chunks_sum_any<BF16>(raw, le, m, block_ref(m, sc), sc));
  if (lane == PTD_WAVE - 1) s_sum[wave] = z;
  __syncthreads();
  if (tid == 0) {
    double t = 0.0;
    for (int w = 0; w < NW; ++w) t += s_sum[w];
    stats[static_cast<size_t>(r) * nblk + blk] = RowStat{m, 0.0f, t};
  }
}

struct SampleArgs {
  const void* logits;
  long long ld;
  int V, T;
  const int32_t* tokens;    // [B][T]
  const int32_t* parent;    // [B][T]
  const int32_t* tree_len;  // [B] or null
  const double* u_node;     // [B][T]
  const double* u_bonus;    // [B][T+1]
  const RowStat* stats;     // [B*(T+1)][nblk] block statistics
  int nblk;
  Scale sc;                 // log2(e) / temperature
  int32_t* accept_len;
  int32_t* accept_nodes;
  int32_t* out_tokens;
  int32_t* dev_status;
};

struct WalkLds {
  int par[PTD_MAX_T], tok[PTD_MAX_T], path[PTD_MAX_T], rej[PTD_MAX_T];
  double p[PTD_MAX_T], u[PTD_MAX_T];
  double rk[PTD_MAX_T + 1];  // row references: the sum of 2^(l c) over row r is
  double rz[PTD_MAX_T + 1];  // rz[r] 2^rk[r]
  uint32_t bits[kMaxVocab / 32];
  double res[kMaxBlocks];    // residual block sums of the terminal's row
  double bscale[kMaxBlocks]; // what the terms of its blocks are multiples of, over 2^rk
  float bm[kMaxBlocks];      // its blocks' largest logits
  double wsum[kWalkWaves];
  RowStat st[kStagedStats];  // every row's block statistics, where they fit
  int first, last, next, depth, nrej, xblk;
  double before, target;
};

// One workgroup per sequence on a handful of CUs: bound by its chain of memory
// round trips and barriers, so loads are issued as early as their addresses are
// known and the block statistics are read once (kept in LDS for the bonus draw
// when (T + 1) * nblk <= kStagedStats).  16 sequences of 64 nodes, 63 blocks a
// row: 12.5 against 16.2 us with one wave per row, a second read of the statistics
// and an LDS look-up and a division per examined child.
template <bool BF16>
__global__ void __launch_bounds__(kWalkThreads) k_verify_sample(SampleArgs a) {
  __shared__ WalkLds L;
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int T = a.T, V = a.V;
  int n = T;
  if (a.tree_len) {
    n = a.tree_len[b];
    n = n < 0 ? 0 : (n > T ? T : n);
  }
  const size_t row0 = static_cast<size_t>(b) * (T + 1);
  auto row_ptr = [&](int r) {
    return static_cast<const char*>(a.logits) + (row0 + r) * a.ld * (BF16 ? 2 : 4);
  };
  int32_t* an = a.accept_nodes + static_cast<size_t>(b) * T;
  int32_t* ot = a.out_tokens + row0;

  // stage the tree and the uniforms; every row's maximum and normalizer from
  // its blocks (loads of both issued together); each node's logit under its
  // parent's row is gathered as soon as the node's own entries have landed
  bool bad = false;
  int my_par = -1, my_tok = -1;
  float my_l = 0.f;
  if (tid < n) {
    my_par = a.parent[static_cast<size_t>(b) * T + tid];
    my_tok = a.tokens[static_cast<size_t>(b) * T + tid];
    L.u[tid] = a.u_node[static_cast<size_t>(b) * T + tid];
  }
  for (int w = tid; w < (V + 31) / 32; w += kWalkThreads) L.bits[w] = 0u;
  // row references and normalizers: 16 lanes per row, 64 rows at a time, four
  // blocks per lane and two rows in flight
  const bool staged = (T + 1) * a.nblk <= kStagedStats;  // uniform
  constexpr int kRowLanes = 16, kRows = kWalkThreads / kRowLanes, kAtOnce = 2, kPer = 4;
  const int gl = tid & (kRowLanes - 1);
  for (int r0 = tid / kRowLanes; r0 <= T; r0 += kAtOnce * kRows) {
    double k[kAtOnce], z[kAtOnce];
#pragma unroll
    for (int j = 0; j < kAtOnce; ++j) {
      k[j] = -INFINITY;
      z[j] = 0.0;
    }
    for (int h0 = 0; h0 < a.nblk; h0 += kPer * kRowLanes) {
      RowStat st[kAtOnce][kPer];
      double kb[kAtOnce][kPer];
#pragma unroll
      for (int j = 0; j < kAtOnce; ++j)
#pragma unroll
        for (int h = 0; h < kPer; ++h) {
          const int r = r0 + j * kRows, x = h0 + h * kRowLanes + gl;
          st[j][h] = RowStat{kLowest, 0.0f, 0.0};
          if (r <= T && x < a.nblk) st[j][h] = a.stats[(row0 + r) * a.nblk + x];
        }
#pragma unroll
      for (int j = 0; j < kAtOnce; ++j) {
#pragma unroll
        for (int h = 0; h < kPer; ++h) kb[j][h] = block_ref(st[j][h].m, a.sc);
        const double kn = fmax(fmax(fmax(kb[j][0], kb[j][1]), fmax(kb[j][2], kb[j][3])), k[j]);
        z[j] *= pow2i(k[j] - kn);
        k[j] = kn;
#pragma unroll
        for (int h = 0; h < kPer; ++h) {
          const int r = r0 + j * kRows, x = h0 + h * kRowLanes + gl;
          z[j] += st[j][h].z * pow2i(kb[j][h] - kn);
          if (staged && r <= T && x < a.nblk) L.st[r * a.nblk + x] = st[j][h];
        }
      }
    }
#pragma unroll
    for (int j = 0; j < kAtOnce; ++j) {
      double kr = k[j];
      kr = fmax(kr, dpp_f64<0x128, 0xF>(kr));  // row_ror 8, 4, 2, 1
      kr = fmax(kr, dpp_f64<0x124, 0xF>(kr));
      kr = fmax(kr, dpp_f64<0x122, 0xF>(kr));
      kr = fmax(kr, dpp_f64<0x121, 0xF>(kr));
      double zr = z[j] * pow2i(k[j] - kr);
      zr += dpp_f64<0x128, 0xF>(zr);
      zr += dpp_f64<0x124, 0xF>(zr);
      zr += dpp_f64<0x122, 0xF>(zr);
      zr += dpp_f64<0x121, 0xF>(zr);
      const int r = r0 + j * kRows;
      if (gl == 0 && r <= T) {
        L.rk[r] = kr;
        L.rz[r] = zr;
      }
    }
  }
  if (tid < n) {
    bad = my_par < -1 || my_par >= tid;
    L.par[tid] = my_par;
    L.tok[tid] = my_tok;
    if (!bad && my_tok >= 0 && my_tok < V) my_l = logit<BF16>(row_ptr(my_par + 1), my_tok);
  }
  if (__syncthreads_or(bad)) {
    if (tid == 0) ptd::report(a.dev_status, PTD_ERR_BAD_TREE);
    for (int i = tid; i <= T; i += kWalkThreads) {
      if (i < T) an[i] = -1;
      ot[i] = -1;
    }
    if (tid == 0) a.accept_len[b] = 0;
    return;
  }
  if (tid < n) {
    const int r = my_par + 1;
    L.p[tid] = (my_tok >= 0 && my_tok < V)
                   ? exp2(scaled(my_l, L.rk[r], a.sc)) / L.rz[r]
                   : 0.0;
  }
  if (tid == 0) {
    L.depth = 0;
    L.nrej = 0;
  }
  __syncthreads();

  // the walk, by wave 0 alone.  At node v the children (nodes c > v with
  // parent v) are listed 64 at a time in index order by a ballot; the
  // decisions then run over them in order with wave-uniform values (token,
  // probability and uniform broadcast from the child's lane): a token
  // already rejected at v counts with p = 0 (a rejected child of this ballot
  // carries it, or, past the first 64 nodes, its bit is set), the child is
  // accepted iff u S < p, else S -= p and its token is rejected (kept in L.rej
  // and marked in the bitmap, cleared when the walk moves on).
  if (wave == 0) {
    int v = -1, depth = 0, nrej = 0;
    for (;;) {
      double S = 1.0;
      int next = -1;
      for (int c0 = v + 1; c0 < n && next < 0; c0 += PTD_WAVE) {
        const int c = c0 + lane;
        const bool kid = c < n && L.par[c] == v;
        uint64_t kb = __ballot(kid), rejected = 0;
        const int t_l = kid ? L.tok[c] : -1;
        const double p_l = kid ? L.p[c] : 0.0;
        const double u_l = kid ? L.u[c] : 2.0;
        while (kb) {  // uniform
          const int src = __builtin_ctzll(kb);
          kb &= kb - 1ull;
          const int t = __builtin_amdgcn_readlane(t_l, src);
          const double p0 = readlane_f64(p_l, src), u = readlane_f64(u_l, src);
          const bool valid = t >= 0 && t < V;
          bool dup = (__ballot(t_l == t) & rejected) != 0;
          if (c0 > v + 1) dup |= valid && ((L.bits[t >> 5] >> (t & 31)) & 1u);
          const double p = dup ? 0.0 : p0;
          if (S > 0.0 && u * S < p) {
            next = c0 + src;
            break;
          }
          S -= p;
          rejected |= 1ull << src;
          if (valid && !dup) {
            if (lane == 0) {
              L.bits[t >> 5] |= 1u << (t & 31);
              L.rej[nrej] = t;
            }
            ++nrej;
          }
        }
      }
      if (next < 0) break;
      // accepted: clear this node's rejections, move to the child
      for (int j = lane; j < nrej; j += PTD_WAVE) {
        const int t = L.rej[j];
        atomicAnd(&L.bits[t >> 5], ~(1u << (t & 31)));
      }
      nrej = 0;
      if (lane == 0) L.path[depth] = next;
      ++depth;
      v = next;
    }
    if (lane == 0) {
      L.depth = depth;
      L.nrej = nrej;
      L.next = v;
    }
  }
  __syncthreads();
  const int v = L.next;

  // the bonus token: inverse CDF of the residual distribution of row v + 1.
  // term(y) = 2^(l_y c - k), formed exactly as in the block sums; the residual
  // block sums (block sum less the rejected terms) locate the block, whose
  // terms are then scanned.
  const int r = v + 1;
  const double kr = L.rk[r];
  const RowStat* bs = a.stats + (row0 + r) * a.nblk;
  const char* rowp = row_ptr(r);
  // block references, scales and sums, and the rejected tokens' terms (their
  // loads issued together, one thread per block / per rejected token)
  const int nrej_t = L.nrej;
  for (int k = tid; k < a.nblk; k += kWalkThreads) {
    const RowStat st = staged ? L.st[r * a.nblk + k] : bs[k];
    const double kb = block_ref(st.m, a.sc), f = pow2i(kb - kr);
    L.bm[k] = st.m;
    L.bscale[k] = block_scale(st.m, kb, a.sc) * f;
    L.res[k] = st.z * f;
  }
  if (tid < nrej_t) {
    const int t = L.rej[tid], k = t / kBlock;
    const float m = staged ? L.st[r * a.nblk + k].m : bs[k].m;
    const double kb = block_ref(m, a.sc);
    L.p[tid] = static_cast<double>(block_term<BF16>(logit<BF16>(rowp, t), m, kb, a.sc)) *
               (block_scale(m, kb, a.sc) * pow2i(kb - kr));
  }
  __syncthreads();
  auto term = [&](int y) -> double {
    const int k = y / kBlock;
    const float m = L.bm[k];
    return static_cast<double>(block_term<BF16>(logit<BF16>(rowp, y), m, block_ref(m, a.sc), a.sc)) * L.bscale[k];
  };
  if (tid == 0)
    for (int j = 0; j < nrej_t; ++j)  // the rejected tokens' terms leave their blocks
      L.res[L.rej[j] / kBlock] -= L.p[j];
  // (usually one turn: what is left of a block's sum may be the rounding of terms
  // that all left it, and such a block is passed over)
  for (;;) {
    if (wave == 0) {
      // running totals over the blocks (fp64 wave scans, two blocks per lane:
      // k = lane and k = 64 + lane); the first block with residual mass whose
      // running total passes the target; if rounding leaves none, the last
      // block with residual mass
      const double r0 = lane < a.nblk ? L.res[lane] : 0.0;
      const double r1 = lane + PTD_WAVE < a.nblk ? L.res[lane + PTD_WAVE] : 0.0;
      const double i0 = wave_incl_scan_f64(r0);
      const double t0 = readlane_f64(i0, PTD_WAVE - 1);
      const double i1 = t0 + wave_incl_scan_f64(r1);
      const double total = readlane_f64(i1, PTD_WAVE - 1);
      const double target = a.u_bonus[row0 + r] * total;
      const uint64_t h0 = __ballot(r0 > 0.0 && i0 > target), h1 = __ballot(r1 > 0.0 && i1 > target);
      const uint64_t m0 = __ballot(r0 > 0.0), m1 = __ballot(r1 > 0.0);
      int xb;
      if (h0 | h1) xb = h0 ? __builtin_ctzll(h0) : PTD_WAVE + __builtin_ctzll(h1);
      else if (m1 | m0) xb = m1 ? 2 * PTD_WAVE - 1 - __builtin_clzll(m1) : PTD_WAVE - 1 - __builtin_clzll(m0);
      else xb = -1;
      // the running total before block xb: the scans' exclusive values (the
      // shuffles run on every lane; lane 0's results are replaced afterwards)
      double e0 = shfl_up_f64(i0, 1);
      double e1 = shfl_up_f64(i1, 1);
      if (lane == 0) {
        e0 = 0.0;
        e1 = t0;
      }
      const int xl = xb < 0 ? 0 : xb & (PTD_WAVE - 1);
      const double b0 = readlane_f64(e0, xl), b1 = readlane_f64(e1, xl);
      if (lane == 0) {
        L.xblk = total > 0.0 ? xb : -1;
        L.before = xb >= PTD_WAVE ? b1 : b0;
        L.target = target;
      }
    }
    __syncthreads();
    const int xb = L.xblk;
    if (xb < 0) {  // no residual mass: every token was rejected
      if (tid == 0) ot[L.depth] = -1;
      break;
    }
    // the block's terms, two consecutive entries per thread, in index order
    const int ya = xb * kBlock + 2 * tid, yb = ya + 1;
    const bool in_a = ya < V && !((L.bits[ya >> 5] >> (ya & 31)) & 1u);
    const bool in_b = yb < V && !((L.bits[yb >> 5] >> (yb & 31)) & 1u);
    const double ea = in_a ? term(ya) : 0.0, eb = in_b ? term(yb) : 0.0;
    const double own = ea + eb;
    const double incl = wave_incl_scan_f64(own);
    double excl = shfl_up_f64(incl, 1);
    if (lane == 0) excl = 0.0;
    if (lane == 63) L.wsum[wave] = incl;
    if (tid == 0) {
      L.first = kWalkThreads;
      L.last = -1;
    }
    __syncthreads();
    double start = L.before;
    for (int w = 0; w < wave; ++w) start += L.wsum[w];
    const double target = L.target;
    // the first thread past the target; if rounding leaves none, the last one with mass
    const uint64_t mass = __ballot(own > 0.0), past = __ballot(own > 0.0 && start + incl > target);
    if (lane == 0 && mass) atomicMax(&L.last, wave * PTD_WAVE + PTD_WAVE - 1 - __builtin_clzll(mass));
    if (lane == 0 && past) atomicMin(&L.first, wave * PTD_WAVE + __builtin_ctzll(past));
    __syncthreads();
    const bool fallback = L.first == kWalkThreads;
    const int pick = fallback ? L.last : L.first;
    if (pick >= 0) {  // uniform
      if (tid == pick) {
        const double cum = start + excl;
        int x;
        if (ea > 0.0 && (!fallback && cum + ea > target)) x = ya;
        else x = eb > 0.0 ? yb : ya;
        ot[L.depth] = x;
      }
      break;
    }
    if (tid == 0) L.res[xb] = 0.0;
    __syncthreads();
  }
  const int depth = L.depth;
  for (int i = tid; i <= T; i += kWalkThreads) {
    if (i < T) an[i] = i < depth ? L.path[i] : -1;
    if (i < depth) ot[i] = L.tok[L.path[i]];
    else if (i > depth) ot[i] = -1;
  }
  if (tid == 0) a.accept_len[b] = depth;
}

}  // namespace

extern "C" size_t ptd_verify_sample_workspace_bytes(int32_t B, int32_t T, int32_t V) {
  if (B < 1 || T < 1 || T > PTD_MAX_T || V < 1 || V > kMaxVocab) return 0;
  const int nblk = (V + kBlock - 1) / kBlock;
  const size_t n = static_cast<size_t>(B) * (T + 1) * nblk * sizeof(RowStat);
  return (n + 255) & ~static_cast<size_t>(255);
}

extern "C" int ptd_verify_sample(const void* logits, ptd_dtype dtype, int32_t V, int64_t ld,
                                 const int32_t* draft_tokens, const int32_t* parent,
                                 const int32_t* tree_len, int32_t B, int32_t T,
                                 double temperature, const double* u_node,
                                 const double* u_bonus, int32_t* accept_len,
                                 int32_t* accept_nodes, int32_t* out_tokens, void* workspace,
                                 size_t workspace_bytes, int32_t* dev_status, void* stream) {
  PTD_RETURN_IF(!logits || !draft_tokens || !parent || !u_node || !u_bonus || !accept_len ||
                    !accept_nodes || !out_tokens,
                PTD_ERR_NULL);
  PTD_RETURN_IF(dtype != PTD_BF16 && dtype != PTD_F32, PTD_ERR_DTYPE);
  PTD_RETURN_IF(B < 1 || T < 1 || T > PTD_MAX_T || V < 1 || V > kMaxVocab || ld < V,
                PTD_ERR_SHAPE);
  PTD_RETURN_IF(!(temperature > 0.0 && temperature < INFINITY), PTD_ERR_SHAPE);
  PTD_RETURN_IF(static_cast<long long>(B) * (T + 1) > 65535, PTD_ERR_SHAPE);  // grid rows
  const size_t need = ptd_verify_sample_workspace_bytes(B, T, V);
  PTD_RETURN_IF(!workspace || workspace_bytes < need, PTD_ERR_WORKSPACE);
  PTD_RETURN_IF(!ptd_aligned(workspace, 16), PTD_ERR_ALIGN);
  hipStream_t st = static_cast<hipStream_t>(stream);
  RowStat* stats = static_cast<RowStat*>(workspace);
  const double c = 1.4426950408889634 / temperature;
  const float c_hi = static_cast<float>(c);
  const Scale sc{c, c_hi, static_cast<float>(c - static_cast<double>(c_hi)), static_cast<float>(-2000.0 / c),
                 static_cast<float>(-200.0 / c), c >= 1.0e-20 && c <= 1.0e30};
  const int R = B * (T + 1);
  const int nblk = (V + kBlock - 1) / kBlock;
  SampleArgs a{logits, ld, V, T, draft_tokens, parent, tree_len, u_node, u_bonus, stats, nblk,
               sc, accept_len, accept_nodes, out_tokens, dev_status};
  // statistics: one wave per block when the call has many blocks (a batch
  // of sequences: 1040 rows x 63 blocks, 50.4 against 85 us), else one
  // workgroup per block (a single sequence's 65-97 rows: 0.8 us shorter)
  const bool wave_stats = static_cast<long long>(R) * nblk >= 8192;
  const dim3 sgrid = wave_stats
      ? dim3((nblk + kStatThreads / PTD_WAVE - 1) / (kStatThreads / PTD_WAVE), R)
      : dim3(nblk, R);
#define PTD_STATS(bf_)                                                                        \
  if (wave_stats)                                                                             \
    hipLaunchKernelGGL(k_block_stats<bf_>, sgrid, dim3(kStatThreads), 0, st, logits, V, ld,   \
                       nblk, sc, stats);                                              \
  else                                                                                        \
    hipLaunchKernelGGL(k_block_stats_wg<bf_>, sgrid, dim3(kStatThreads), 0, st, logits, V,    \
                       ld, nblk, sc, stats);                                          \
  hipLaunchKernelGGL(k_verify_sample<bf_>, dim3(B), dim3(kWalkThreads), 0, st, a);
  if (dtype == PTD_BF16) {
    PTD_STATS(true)
  } else {
    PTD_STATS(false)
  }
#undef PTD_STATS
  return ptd_launch_status();
}
