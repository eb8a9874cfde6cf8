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
//                    block maximum m_b and
//                    z_b = sum exp((l - m_b) / temperature) over the block,
//                    each term an fp32 exponential with its argument's
//                    rounding compensated (~1.2e-7 relative), added in fp64.
//   k_verify_sample  one workgroup of 1024 threads per sequence.  Each row's
//                    k = max_b k_b and normalizer z = sum_b z_b 2^(k_b - k)
//                    (exact scalings) are formed in LDS; the tree, the uniforms and every
//                    node's probability under its parent's row (numerator in
//                    fp64) are staged.  Each level of the walk lists the
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
__device__ __forceinline__ double shfl_xor_f64(double x, int d) {
  const uint64_t u = __double_as_longlong(x);
  const uint32_t lo = __shfl_xor(static_cast<uint32_t>(u), d, PTD_WAVE);
  const uint32_t hi = __shfl_xor(static_cast<uint32_t>(u >> 32), d, PTD_WAVE);
  return __longlong_as_double(static_cast<long long>((static_cast<uint64_t>(hi) << 32) | lo));
}

// Sum over a block (or row) of 2^(l c) = z 2^k, c = log2(e) / temperature and k
// an integer within one of the largest l c (powers of two rescale z exactly).
struct RowStat {
  double k, z;
};

// c = log2(e) / temperature as an fp64 value and as c_hi + c_lo in fp32
struct Scale {
  double c;
  float c_hi, c_lo;
};

// Blocks whose largest |l c| is within kFastRange take the fp32 term below.
constexpr float kFastRange = 800.0f;
constexpr float kGrid = 3072.0f;  // 1.5 * 2^11: adding it rounds |y| < 1024 to multiples of 2^-12
// Integer reference of a block (or of the terms of one) from its largest logit;
// a block of -inf only gets a finite one, its terms all 0.
__device__ __forceinline__ double block_ref(float m, const Scale& sc) {
  return fmax(rint(static_cast<double>(m) * sc.c), -1.0e300);
}
__device__ __forceinline__ bool fast_ref(double k) { return fabs(k) <= kFastRange; }
// 2^(l c - k) in fp32 for |k| <= kFastRange.  l c is rounded to a multiple of
// 2^-12 by one FMA, so the subtractions of kGrid and of k are exact; the rest e
// of l c (at most 2^-13, found by two FMAs) enters to first order (second order
// below 6e-9).  The term is within about one ulp of v_exp_f32 (~1.2e-7 relative)
// of the exact value; it is 0 far below the reference, and NaN where l c
// overflows (l = -inf, the type's lowest value): the callers then take
// exp_term_any.
__device__ __forceinline__ void exp_parts(float l, float kf, const Scale& sc, float& p, float& e) {
  const float t = fmaf(l, sc.c_hi, kGrid);
  const float y = t - kGrid;
  e = fmaf(l, sc.c_lo, fmaf(l, sc.c_hi, -y));
  p = __builtin_amdgcn_exp2f(y - kf);
}
constexpr float kLn2 = 0.69314718f;
__device__ __forceinline__ float exp_term(float l, float kf, const Scale& sc) {
  float p, e;
  exp_parts(l, kf, sc, p, e);
  return fmaf(p, e * kLn2, p);
}
// Sum of two terms, the correction applied once.  k_block_stats is bound by its
// vector instructions, 11 per entry here (an exponential counted as two) against
// 19 with (l - m) c, the difference kept in two parts.
__device__ __forceinline__ float exp_pair(float l0, float l1, float kf, const Scale& sc) {
  float p0, e0, p1, e1;
  exp_parts(l0, kf, sc, p0, e0);
  exp_parts(l1, kf, sc, p1, e1);
  return fmaf(fmaf(p1, e1, p0 * e0), kLn2, p0 + p1);
}
// The same for any reference (logits or temperatures far from ordinary ones).
__device__ __noinline__ double exp_term_any(float l, double k, double c) {
  return exp2(static_cast<double>(l) * c - k);
}
__device__ __forceinline__ double term64(float l, double k, const Scale& sc) {
  if (fast_ref(k)) {
    const float t = exp_term(l, static_cast<float>(k), sc);
    if (t == t) return static_cast<double>(t);
  }
  return exp_term_any(l, k, sc.c);
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
// Maximum of the entries of a block by plain loads (every lane gets it).
template <bool BF16>
__device__ __noinline__ float slow_max(const void* row, int y0, int y1, int lane) {
  float m = -INFINITY;
  for (int y = y0 + lane; y < y1; y += PTD_WAVE) m = fmaxf(m, logit<BF16>(row, y));
  return ptd::wave_max(m);
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
  float m = le;
#pragma unroll
  for (int j = 0; j < CPL; ++j) {
    float x[E];
    chunk_vals<BF16>(raw[j], x);
#pragma unroll
    for (int e = 0; e < E; e += 2) m = max3(x[e], x[e + 1], m);
  }
  m = wave_max_uniform(m);
  if (!(m > kNone)) m = slow_max<BF16>(row, y0, y1, lane);  // uniform; padding taken for an entry
  const double k = block_ref(m, sc);
  double z = __builtin_nan("");
  if (fast_ref(k)) {  // uniform
    const float kf = static_cast<float>(k);
    z = static_cast<double>(exp_term(le, kf, sc));
#pragma unroll
    for (int j = 0; j < CPL; ++j) {
      float x[E];
      chunk_vals<BF16>(raw[j], x);
#pragma unroll
      for (int e = 0; e < E; e += 2)  // pairs added in fp32 (one rounding, 2^-24), then fp64
        z += static_cast<double>(exp_pair(x[e], x[e + 1], kf, sc));
    }
  }
  if (__any(!(z == z))) {  // uniform: far logits, or masks that overflow l c
    z = 0.0;
    for (int y = y0 + lane; y < y1; y += PTD_WAVE) z += exp_term_any(logit<BF16>(row, y), k, sc.c);
  }
  z = wave_incl_scan_f64(z);
  if (lane == PTD_WAVE - 1) stats[static_cast<size_t>(r) * nblk + blk] = RowStat{k, z};
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
  float x[CPT][E];
  bool have[CPT];
#pragma unroll
  for (int j = 0; j < CPT; ++j) {
    const int c = tid + j * kStatThreads;
    have[j] = c < sp.nch;
    if (have[j]) chunk_vals<BF16>(sp.chunks[c], x[j]);
  }
  const float le = sp.edge >= 0 ? logit<BF16>(row, sp.edge) : -INFINITY;
  float m = le;
#pragma unroll
  for (int j = 0; j < CPT; ++j)
    if (have[j])
#pragma unroll
      for (int e = 0; e < E; e += 2) m = max3(x[j][e], x[j][e + 1], m);
  m = wave_max_uniform(m);
  if (lane == 0) s_max[wave] = m;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < NW; ++w) m = fmaxf(m, s_max[w]);
  const double k = block_ref(m, sc);
  double z = __builtin_nan("");
  if (fast_ref(k)) {  // uniform
    const float kf = static_cast<float>(k);
    z = sp.edge >= 0 ? static_cast<double>(exp_term(le, kf, sc)) : 0.0;
#pragma unroll
    for (int j = 0; j < CPT; ++j)
      if (have[j])
#pragma unroll
        for (int e = 0; e < E; e += 2)  // pairs added in fp32 (one rounding, 2^-24), then fp64
          z += static_cast<double>(exp_pair(x[j][e], x[j][e + 1], kf, sc));
  }
  // a wave with far logits or masks redoes its own entries: its chunks and edges
  if (__any(!(z == z))) {
    z = sp.edge >= 0 ? exp_term_any(le, k, sc.c) : 0.0;
#pragma unroll
    for (int j = 0; j < CPT; ++j)
      if (have[j])
#pragma unroll 1
        for (int e = 0; e < E; ++e) z += exp_term_any(logit<BF16>(sp.chunks + tid + j * kStatThreads, e), k, sc.c);
  }
  z = wave_incl_scan_f64(z);
  if (lane == PTD_WAVE - 1) s_sum[wave] = z;
  __syncthreads();
  if (tid == 0) {
    double t = 0.0;
    for (int w = 0; w < NW; ++w) t += s_sum[w];
    stats[static_cast<size_t>(r) * nblk + blk] = RowStat{k, t};
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
  int par[PTD_MAX_T], tok[PTD_MAX_T], kids[PTD_MAX_T], path[PTD_MAX_T], rej[PTD_MAX_T];
  double p[PTD_MAX_T], u[PTD_MAX_T];
  double rk[PTD_MAX_T + 1];  // row references: the sum of 2^(l c) over row r is
  double rz[PTD_MAX_T + 1];  // rz[r] 2^rk[r]
  uint32_t bits[kMaxVocab / 32];
  double res[kMaxBlocks];    // residual block sums of the terminal's row
  double bscale[kMaxBlocks]; // 2^(k_b - k) of the terminal's row
  double bk[kMaxBlocks];     // its block references
  double wsum[kWalkWaves];
  RowStat st[kStagedStats];  // every row's block statistics, where they fit
  int first, last, next, depth, nrej, xblk;
  double before, target;
};

// One workgroup per sequence on a handful of CUs: bound by its chain of memory
// round trips and barriers, so loads are issued as early as their addresses are
// known and the block statistics are read once (kept in LDS for the bonus draw
// when (T + 1) * nblk <= kStagedStats).  16 sequences of 64 nodes, 63 blocks a
// row: @@ against 16.2 us with one wave per row, a second read of the statistics
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
#pragma unroll
      for (int j = 0; j < kAtOnce; ++j)
#pragma unroll
        for (int h = 0; h < kPer; ++h) {
          const int r = r0 + j * kRows, x = h0 + h * kRowLanes + gl;
          st[j][h] = RowStat{-INFINITY, 0.0};
          if (r <= T && x < a.nblk) st[j][h] = a.stats[(row0 + r) * a.nblk + x];
        }
#pragma unroll
      for (int j = 0; j < kAtOnce; ++j) {
        const double kn = fmax(fmax(fmax(st[j][0].k, st[j][1].k), fmax(st[j][2].k, st[j][3].k)), k[j]);
        z[j] *= pow2i(k[j] - kn);
        k[j] = kn;
#pragma unroll
        for (int h = 0; h < kPer; ++h) {
          const int r = r0 + j * kRows, x = h0 + h * kRowLanes + gl;
          z[j] += st[j][h].z * pow2i(st[j][h].k - kn);
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
                   ? exp2(static_cast<double>(my_l) * a.sc.c - L.rk[r]) / L.rz[r]
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
  // term(y) = 2^(l_y c - k_b) * 2^(k_b - k) for y in block b, exactly as the
  // block sums were formed; the residual block sums (block sum less
  // the rejected terms) locate the block, whose terms are then scanned.
  const int r = v + 1;
  const double kr = L.rk[r];
  const RowStat* bs = a.stats + (row0 + r) * a.nblk;
  const char* rowp = row_ptr(r);
  // block references, scales and sums, and the rejected tokens' terms (their
  // loads issued together, one thread per block / per rejected token)
  const int nrej_t = L.nrej;
  for (int k = tid; k < a.nblk; k += kWalkThreads) {
    const RowStat st = staged ? L.st[r * a.nblk + k] : bs[k];
    const double f = pow2i(st.k - kr);
    L.bk[k] = st.k;
    L.bscale[k] = f;
    L.res[k] = st.z * f;
  }
  if (tid < nrej_t) {
    const int t = L.rej[tid], k = t / kBlock;
    const double kb = staged ? L.st[r * a.nblk + k].k : bs[k].k;
    L.p[tid] = term64(logit<BF16>(rowp, t), kb, a.sc) * pow2i(kb - kr);
  }
  __syncthreads();
  auto term = [&](int y) -> double {
    const int k = y / kBlock;
    return term64(logit<BF16>(rowp, y), L.bk[k], a.sc) * L.bscale[k];
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
  const Scale sc{c, c_hi, static_cast<float>(c - static_cast<double>(c_hi))};
  const int R = B * (T + 1);
  const int nblk = (V + kBlock - 1) / kBlock;
  SampleArgs a{logits, ld, V, T, draft_tokens, parent, tree_len, u_node, u_bonus, stats, nblk,
               sc, accept_len, accept_nodes, out_tokens, dev_status};
  // statistics: one wave per block when the call has many blocks (a batch
  // of sequences: 1040 rows x 63 blocks, 63.6 against 85 us), else one
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
