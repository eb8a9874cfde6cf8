// Depth control of the draft forest and the value-keyed candidate pool.
//
// Sec. 3.1 "Overhead Constraints" (Stepping Mechanism) and Alg. 1 step 3:
// when a sub-tree is deeper than d_max, its earliest-added (lowest-index)
// child's sub-tree replaces it and the other branches are pruned, repeatedly,
// so a chain keeps its last d_max nodes.  Sec. 3.1 "Draft Extraction via
// Merging" and Alg. 1 steps 1 and 4: every sub-tree of the draft is merged by
// M into the pool tree keyed by its root's token; the candidate tree of the
// next step is the pool tree keyed by the last committed token.
//
// Draft trees have at most 128 nodes and pool trees at most 129 (their root
// included):
//   k_step_prune     one wave per sequence: ancestor sets by pointer doubling,
//                    sub-tree depths, the new root of every sub-tree along its
//                    chain of lowest-index children, and breadth-first
//                    renumbering of the kept forest level by level.
//   k_pool_merge     several waves per sequence, each merging some of the
//                    touched trees in registers.  Every draft node's token is
//                    looked up in the hash table (token -> tree), the missing
//                    tokens get new trees in index order of their first
//                    occurrence (while there is room).  A tree takes the
//                    sub-trees whose root carries its token in index order of
//                    the roots, a sub-tree's nodes in index order (the trees
//                    are independent).  The appended nodes and node counts are
//                    written back (a merge never changes a stored node); the
//                    last wave to have read the table inserts the new tokens.
//   k_pool_retrieve  one wave per sequence: 64 hash slots from the token's home
//                    slot in one load, the tree's nodes three per lane,
//                    breadth-first order by levels.
//
// Pool layout per sequence (ptd_pool_bytes): int32 ntrees, int32
// arrivals (0 between calls), padded to 16 bytes; int32 slot_key[H]; int32 slot_tree[H] (-1 empty); int32 count[e_max];
// int2 node[e_max][n_cap] = (token, parent index in the tree; -1 at the root,
// which is node 0).  H is the power of two >= 2 e_max (at least 64).  Nodes
// of a tree are stored in insertion order, so a parent precedes its children.
#include <algorithm>

#include "ptd_common.hpp"

namespace {

constexpr int kMaxNodes = 128;            // draft nodes per sequence
constexpr int kMaxCap = kMaxNodes + 1;    // pool tree capacity, root included
constexpr int kMaxTrees = 2048;           // pool trees per sequence
constexpr int kInitThreads = 256;
constexpr int kDeadNode = 1 << 20;        // depth of a node without a path to its tree's root

struct PoolGeom {
  int e_max, n_cap, H, hbits;
  size_t seq_bytes, off_key, off_tree, off_count, off_node;
};

inline bool pool_geom(int e_max, int n_cap, PoolGeom* g) {
  if (e_max < 1 || e_max > kMaxTrees || n_cap < 1 || n_cap > kMaxCap) return false;
  int H = 64, hb = 6;
  while (H < 2 * e_max) {
    H <<= 1;
    ++hb;
  }
  g->e_max = e_max;
  g->n_cap = n_cap;
  g->H = H;
  g->hbits = hb;
  g->off_key = 16;
  g->off_tree = g->off_key + 4 * static_cast<size_t>(H);
  g->off_count = g->off_tree + 4 * static_cast<size_t>(H);
  g->off_node = (g->off_count + 4 * static_cast<size_t>(e_max) + 15) & ~static_cast<size_t>(15);
  g->seq_bytes = (g->off_node + 8 * static_cast<size_t>(e_max) * n_cap + 255) & ~static_cast<size_t>(255);
  return true;
}

struct PoolView {
  int32_t* ntrees;
  int32_t* key;
  int32_t* tree;
  int32_t* count;
  int2* node;
};
__device__ __forceinline__ PoolView view(void* pool, const PoolGeom& g, int b) {
  char* base = static_cast<char*>(pool) + static_cast<size_t>(b) * g.seq_bytes;
  return PoolView{reinterpret_cast<int32_t*>(base), reinterpret_cast<int32_t*>(base + g.off_key),
                  reinterpret_cast<int32_t*>(base + g.off_tree),
                  reinterpret_cast<int32_t*>(base + g.off_count),
                  reinterpret_cast<int2*>(base + g.off_node)};
}

__device__ __forceinline__ int home_slot(int token, int hbits) {
  return static_cast<int>((static_cast<uint32_t>(token) * 0x9E3779B1u) >> (32 - hbits));
}

__device__ __forceinline__ uint64_t below_mask(int lane) { return (1ull << lane) - 1ull; }

// ---------------------------------------------------------------------------
// one wave per tree: node 64 x + lane in slot x of its lane (NW = 1: trees of up
// to 64 nodes, 2: up to 128), node sets as NW words
// ---------------------------------------------------------------------------
// r[x] of node i (i: per lane; uniform)
template <int NW>
__device__ __forceinline__ int node_get(const int (&r)[NW], int i) {
  int a = __shfl(r[0], i & 63, PTD_WAVE);
  if constexpr (NW == 2) {
    const int c = __shfl(r[1], i & 63, PTD_WAVE);
    a = i >= 64 ? c : a;
  }
  return a;
}
template <int NW>
__device__ __forceinline__ int node_read(const int (&r)[NW], int i) {
  const int a = __builtin_amdgcn_readlane(r[0], i & 63);
  if constexpr (NW == 1) return a;
  else return i >= 64 ? __builtin_amdgcn_readlane(r[NW - 1], i & 63) : a;
}

// Ancestor-or-self sets (word w of a node's set: nodes 64 w ..) by pointer doubling.
template <int NW>
__device__ __forceinline__ void ancestor_sets(const bool (&live)[NW], const int (&par)[NW],
                                              uint64_t (&anc)[NW][NW]) {
  const int lane = threadIdx.x & (PTD_WAVE - 1);
  int jump[NW];
#pragma unroll
  for (int x = 0; x < NW; ++x) {
#pragma unroll
    for (int w = 0; w < NW; ++w) anc[x][w] = live[x] && w == x ? 1ull << lane : 0ull;
    jump[x] = par[x];
  }
  for (;;) {
    bool more = false;
#pragma unroll
    for (int x = 0; x < NW; ++x) more |= jump[x] >= 0;
    if (!__any(more)) break;
    int lo[NW], hi[NW], nj[NW];
    uint64_t na[NW][NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) {
#pragma unroll
      for (int x = 0; x < NW; ++x) {
        lo[x] = static_cast<int>(static_cast<uint32_t>(anc[x][w]));
        hi[x] = static_cast<int>(static_cast<uint32_t>(anc[x][w] >> 32));
      }
#pragma unroll
      for (int x = 0; x < NW; ++x) {
        const int a = max(jump[x], 0);
        na[x][w] = static_cast<uint64_t>(static_cast<uint32_t>(node_get<NW>(lo, a))) |
                   (static_cast<uint64_t>(static_cast<uint32_t>(node_get<NW>(hi, a))) << 32);
      }
    }
#pragma unroll
    for (int x = 0; x < NW; ++x) nj[x] = node_get<NW>(jump, max(jump[x], 0));
#pragma unroll
    for (int x = 0; x < NW; ++x)
      if (jump[x] >= 0) {
#pragma unroll
        for (int w = 0; w < NW; ++w) anc[x][w] |= na[x][w];
        jump[x] = nj[x];
      }
  }
}

// Members of the set m below node i.
template <int NW>
__device__ __forceinline__ int count_below(const uint64_t (&m)[NW], int i) {
  if constexpr (NW == 1) return __popcll(m[0] & below_mask(i & 63));
  else return i < 64 ? __popcll(m[0] & below_mask(i & 63))
                     : __popcll(m[0]) + __popcll(m[NW - 1] & below_mask(i & 63));
}

// Exclusive prefix sum over the lanes, and the total: row_shr 1, 2, 4, 8 within
// each row of 16 lanes, then the rows' totals by row_bcast 15 and 31.
__device__ __forceinline__ int wave_excl_sum(int c, int* total) {
  int x = c;
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);
  *total = __builtin_amdgcn_readlane(x, 63);
  return x - c;
}

// ---------------------------------------------------------------------------
// stepping: one wave per sequence.  Bound by its chain of dependent LDS and
// shuffle steps: 4.2 us for 16 trees of 64 nodes (11.0 with a thread per node and
// a barrier at every step, whose level ranks read every member's key).
// ---------------------------------------------------------------------------
template <int NW>
__global__ void __launch_bounds__(PTD_WAVE)
k_step_prune(const int32_t* __restrict__ parent, const int32_t* __restrict__ tokens,
             const int32_t* __restrict__ tree_len, int T, int d_max, int T_max,
             int32_t* __restrict__ parent_next, int32_t* __restrict__ tokens_next,
             int32_t* __restrict__ tree_len_next, int32_t* dev_status) {
  constexpr int N = PTD_WAVE * NW;
  __shared__ uint64_t s_cm[N][NW];  // children
  __shared__ int s_deep[N];         // depth of the deepest node below or at each
  __shared__ int s_fc[N];           // lowest-index child
  __shared__ int s_rootof[N];       // new roots: the old root they replace
  __shared__ int s_out[N];          // new number
  __shared__ int s_cnt[N];          // by position in a level: children, then first child's number
  const int lane = threadIdx.x, b = blockIdx.x;
  int n = T;
  if (tree_len) {
    n = tree_len[b];
    n = n < 0 ? 0 : (n > T ? T : n);
  }
  int32_t* pn = parent_next + static_cast<size_t>(b) * T_max;
  int32_t* tn = tokens_next + static_cast<size_t>(b) * T_max;
  int par[NW], tok[NW];
  bool live[NW], bad = false;
#pragma unroll
  for (int x = 0; x < NW; ++x) {
    const int v = 64 * x + lane;
    const int p = v < T ? parent[static_cast<size_t>(b) * T + v] : -1;
    tok[x] = v < T ? tokens[static_cast<size_t>(b) * T + v] : -1;
    live[x] = v < n;
    par[x] = live[x] ? p : -1;
    bad |= par[x] < -1 || par[x] >= v;
    s_deep[v] = 0;
    s_fc[v] = N;
    s_rootof[v] = -1;
#pragma unroll
    for (int w = 0; w < NW; ++w) s_cm[v][w] = 0ull;
  }
  if (__any(bad)) {
    if (lane == 0) {
      ptd::report(dev_status, PTD_ERR_BAD_TREE);
      tree_len_next[b] = 0;
    }
    for (int t = lane; t < T_max; t += PTD_WAVE) {
      pn[t] = -1;
      tn[t] = -1;
    }
    return;
  }
  uint64_t anc[NW][NW];
  ancestor_sets<NW>(live, par, anc);
  __syncthreads();  // (one wave: orders the LDS accesses)
  int dep[NW];
#pragma unroll
  for (int x = 0; x < NW; ++x) {
    dep[x] = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) dep[x] += __popcll(anc[x][w]);
    if (par[x] >= 0) {
      atomicOr(reinterpret_cast<unsigned long long*>(&s_cm[par[x]][x]), 1ull << lane);
      atomicMin(&s_fc[par[x]], 64 * x + lane);
    }
  }
  __syncthreads();
  // The deepest level below a node is a leaf's, and among a node's children the
  // first or one below it reaches at least as deep as any leaf: only leaves that
  // are a first child (or a root) enter theirs.  s_deep is read along first
  // children alone.  (Every node entering its own cost a chain of 128 nodes 8256
  // LDS atomics, most of them to one address: 1024 of them 45 us, now 26.6.)
#pragma unroll
  for (int x = 0; x < NW; ++x) {
    const int v = 64 * x + lane;
    const bool enters = live[x] && s_fc[v] == N && (par[x] < 0 || s_fc[par[x]] == v);
#pragma unroll
    for (int w = 0; w < NW; ++w)
      for (uint64_t m = enters ? anc[x][w] : 0ull; m; m &= m - 1ull)
        atomicMax(&s_deep[64 * w + __builtin_ctzll(m)], dep[x]);
  }
  __syncthreads();
  // every old root steps down its lowest-index children while too deep
  uint64_t old_roots[NW], roots[NW], keep[NW];
#pragma unroll
  for (int x = 0; x < NW; ++x) {
    const bool root = live[x] && par[x] < 0;
    old_roots[x] = __ballot(root);
    if (root) {
      int v = 64 * x + lane;
      for (int d = 1; s_deep[v] - d + 1 > d_max; ++d) v = s_fc[v];
      s_rootof[v] = 64 * x + lane;
    }
  }
  __syncthreads();
  int rootof[NW], nd[NW];
#pragma unroll
  for (int x = 0; x < NW; ++x) {
    rootof[x] = s_rootof[64 * x + lane];
    roots[x] = __ballot(rootof[x] >= 0);
  }
  bool kept[NW];
#pragma unroll
  for (int x = 0; x < NW; ++x) {
    kept[x] = false;
#pragma unroll
    for (int w = 0; w < NW; ++w) kept[x] |= (anc[x][w] & roots[w]) != 0ull;
    keep[x] = __ballot(kept[x]);
  }
  int total = 0, hi = 0;
#pragma unroll
  for (int x = 0; x < NW; ++x) {
    total += __popcll(keep[x]);
    hi += __popcll(old_roots[x]);  // one new root each
    nd[x] = 0;  // depth in the kept forest
#pragma unroll
    for (int w = 0; w < NW; ++w) nd[x] += __popcll(anc[x][w] & keep[w]);
  }
  // breadth-first numbering: level 1 in the order of the old roots, then level by
  // level the children (all kept) of a node in index order: a level's nodes write
  // their child counts at their positions, whose prefix sums number the children
  int out[NW], pout[NW], sib[NW], nch[NW];
#pragma unroll
  for (int x = 0; x < NW; ++x) {
    out[x] = pout[x] = -1;
    if (rootof[x] >= 0) out[x] = count_below<NW>(old_roots, rootof[x]);
    uint64_t cm[NW], own[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      cm[w] = s_cm[max(par[x], 0)][w];
      own[w] = s_cm[64 * x + lane][w];
    }
    sib[x] = count_below<NW>(cm, 64 * x + lane);
    nch[x] = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) nch[x] += __popcll(own[w]);
    if (out[x] >= 0) s_out[64 * x + lane] = out[x];
  }
  for (int L = 1, lo = 0; hi < total; ++L) {  // uniform; every level has children up to the last
    const int len = hi - lo;
#pragma unroll
    for (int x = 0; x < NW; ++x)
      if (kept[x] && nd[x] == L) s_cnt[out[x] - lo] = nch[x];
    __syncthreads();
    int run = hi;
#pragma unroll
    for (int x = 0; x < NW; ++x) {
      const int pos = 64 * x + lane;
      int sum;
      const int e = wave_excl_sum(pos < len ? s_cnt[pos] : 0, &sum);
      if (pos < len) s_cnt[pos] = run + e;
      run += sum;
    }
    __syncthreads();
#pragma unroll
    for (int x = 0; x < NW; ++x)
      if (kept[x] && nd[x] == L + 1) {
        pout[x] = s_out[par[x]];
        out[x] = s_cnt[pout[x] - lo] + sib[x];
        s_out[64 * x + lane] = out[x];
      }
    lo = hi;
    hi = run;
    __syncthreads();
  }
#pragma unroll
  for (int x = 0; x < NW; ++x)
    if (kept[x] && out[x] < T_max) {
      pn[out[x]] = pout[x];
      tn[out[x]] = tok[x];
    }
  for (int t = total + lane; t < T_max; t += PTD_WAVE) {
    pn[t] = -1;
    tn[t] = -1;
  }
  if (lane == 0) tree_len_next[b] = min(total, T_max);
}

// ---------------------------------------------------------------------------
// pool
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(kInitThreads) k_pool_init(void* pool, PoolGeom g) {
  const int b = blockIdx.x;
  PoolView P = view(pool, g, b);
  for (int i = threadIdx.x; i < g.H; i += kInitThreads) {
    P.key[i] = 0;
    P.tree[i] = -1;
  }
  if (threadIdx.x == 0) {
    P.ntrees[0] = 0;
    P.ntrees[1] = 0;  // arrivals of a merge's waves
  }
}

// Merge.  One wave per share of a sequence's touched pool trees, X waves per
// sequence, no LDS and no barrier: node 64 x + lane of the draft in slot x of its
// lane (NW = 1: drafts of up to 64 nodes), node 64 q + lane of the pool tree at
// hand in register q.  Every wave looks all tokens up and numbers the new trees
// (the same in each); it then merges the touched trees of its share one after the
// other, the next one's records loading meanwhile.  A merge step (one node of one
// sub-tree) finds the child by a ballot over the tree's nodes.  Nobody may change
// the hash table while another wave still reads it: each wave counts itself in
// (word 1 of the sequence's header) once its look-ups are done, and the last one
// inserts the new tokens and sets the counter back.
// Bound by latency: token, hash and tree loads (three round trips), then about
// 0.1 us per merge step of a wave.  16 sequences of 64 nodes into 65-node trees:
// 10.3 us per call; one workgroup per sequence, tables and trees staged in LDS and
// one thread per tree, took 28.3 (drafts of 96 nodes into 97-node trees 17.1
// against 47.6).
constexpr int kTreeRegs = (kMaxCap + PTD_WAVE - 1) / PTD_WAVE;

// lowest node of a set, taken out of it; -1: empty (uniform)
template <int NW>
__device__ __forceinline__ int pop_node(uint64_t (&m)[NW]) {
  if (m[0]) {
    const int v = __builtin_ctzll(m[0]);
    m[0] &= m[0] - 1ull;
    return v;
  }
  if (NW == 2 && m[NW - 1]) {
    const int v = 64 + __builtin_ctzll(m[NW - 1]);
    m[NW - 1] &= m[NW - 1] - 1ull;
    return v;
  }
  return -1;
}

// Q: registers per lane that hold a tree's nodes (n_cap <= 64 Q)
template <int NW, int Q>
__global__ void __launch_bounds__(PTD_WAVE)
k_pool_merge(void* pool, PoolGeom g, const int32_t* __restrict__ parent,
             const int32_t* __restrict__ tokens, const int32_t* __restrict__ tree_len, int T,
             int X, int32_t* dev_status) {
  // Share by share over the sequences: workgroups go round-robin to the XCDs, so
  // the first shares, which hold the largest trees, spread over them and start
  // first (one token in 256 drafts of 128 nodes: 3290 us per call sequence by
  // sequence, where 32 shares put every first one on the same XCD, now 1163).
  const int B = static_cast<int>(gridDim.x) / X;
  const int share = static_cast<int>(blockIdx.x) / B, b = static_cast<int>(blockIdx.x) - share * B;
  const int lane = threadIdx.x;
  PoolView P = view(pool, g, b);
  int n = T;
  if (tree_len) {
    n = tree_len[b];
    n = n < 0 ? 0 : (n > T ? T : n);
  }
  int par[NW], tok[NW];
  bool live[NW], bad = false;
#pragma unroll
  for (int x = 0; x < NW; ++x) {
    const int v = 64 * x + lane;
    live[x] = v < n;
    par[x] = live[x] ? parent[static_cast<size_t>(b) * T + v] : -1;
    tok[x] = live[x] ? tokens[static_cast<size_t>(b) * T + v] : 0;
    bad |= par[x] < -1 || par[x] >= v;
  }
  const int ntrees0 = min(max(*P.ntrees, 0), g.e_max);
  if (__any(bad)) {
    if (share == 0 && lane == 0) ptd::report(dev_status, PTD_ERR_BAD_TREE);
    return;  // the pool is left as it was
  }

  // look-ups, four slots of every node at a time; the first ones load while the
  // first node (index order) of every token is found
  constexpr int kProbe = 4;
  const int H = g.H;
  int ptree[NW][kProbe], pkey[NW][kProbe], home[NW];
  auto probe = [&](int k0) __attribute__((always_inline)) {
#pragma unroll
    for (int x = 0; x < NW; ++x)
#pragma unroll
      for (int q = 0; q < kProbe; ++q) {
        const int s = (home[x] + k0 + q) & (H - 1);
        ptree[x][q] = P.tree[s];
        pkey[x][q] = P.key[s];
      }
  };
#pragma unroll
  for (int x = 0; x < NW; ++x) home[x] = home_slot(tok[x], g.hbits);
  probe(0);
  int first[NW];
#pragma unroll
  for (int x = 0; x < NW; ++x) first[x] = 64 * x + lane;
#pragma unroll 4
  for (int u = n - 1; u >= 0; --u) {  // downwards: the lowest match stays
    const int tu = node_read<NW>(tok, u);
#pragma unroll
    for (int x = 0; x < NW; ++x) first[x] = tok[x] == tu ? u : first[x];
  }
  int e[NW];
  bool open[NW];
#pragma unroll
  for (int x = 0; x < NW; ++x) {
    e[x] = -1;
    open[x] = live[x];
  }
  for (int k0 = 0;;) {
    bool more = false;
#pragma unroll
    for (int x = 0; x < NW; ++x) {
#pragma unroll
      for (int q = 0; q < kProbe; ++q) {
        const int tr = ptree[x][q];
        const bool hit = tr >= 0 && pkey[x][q] == tok[x];
        // an id out of range (a pool not initialised) reads as absent
        if (open[x] && hit) e[x] = tr < g.e_max ? tr : -1;
        open[x] = open[x] && tr >= 0 && !hit;
      }
      more |= open[x];
    }
    k0 += kProbe;
    if (!__any(more) || k0 >= H) break;
    probe(k0);
  }
  // this wave has read the table and the tree count
  int* arrivals = P.ntrees + 1;
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  int arrived = 0;
  if (lane == 0) arrived = atomicAdd(arrivals, 1);

  // new trees for the missing tokens, in index order of their first node
  int newid[NW];
  bool newfirst[NW], created[NW];
  int nnew = 0;
#pragma unroll
  for (int x = 0; x < NW; ++x) {
    newfirst[x] = live[x] && e[x] < 0 && first[x] == 64 * x + lane;
    const uint64_t m = __ballot(newfirst[x]);
    const int id = ntrees0 + nnew + __popcll(m & below_mask(lane));
    newid[x] = newfirst[x] && id < g.e_max ? id : -1;
    nnew += __popcll(m);
  }
#pragma unroll
  for (int x = 0; x < NW; ++x) {
    const int id = node_get<NW>(newid, first[x]);
    created[x] = live[x] && e[x] < 0 && id >= 0;
    if (created[x]) e[x] = id;
  }
  // touched trees in order of first use, every X-th one this wave's
  uint64_t mine[NW], isnew[NW];
  int nd = 0;
#pragma unroll
  for (int x = 0; x < NW; ++x) {
    const bool use = live[x] && e[x] >= 0 && first[x] == 64 * x + lane;
    const uint64_t m = __ballot(use);
    const int j = nd + __popcll(m & below_mask(lane));
    mine[x] = __ballot(use && j % X == share);
    isnew[x] = __ballot(created[x]);
    nd += __popcll(m);
  }
  uint64_t anc[NW][NW];
  ancestor_sets<NW>(live, par, anc);

  const int n_cap = g.n_cap;
  int2 rec[Q];
  int rec_cnt = 0;
  auto is_new = [&](int f) __attribute__((always_inline)) {
    const uint64_t m0 = isnew[0], m1 = isnew[NW - 1];
    return (((f >= 64 ? m1 : m0) >> (f & 63)) & 1ull) != 0;
  };
  auto load_tree = [&](int f) __attribute__((always_inline)) {
    const int et = node_read<NW>(e, f);
    rec_cnt = 0;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int k = 64 * q + lane;
      rec[q] = make_int2(0, -1);
      if (!is_new(f) && k < n_cap) rec[q] = P.node[static_cast<size_t>(et) * n_cap + k];
    }
    if (!is_new(f)) rec_cnt = P.count[et];
  };
  int f = pop_node<NW>(mine);  // first node of the tree's token
  if (f >= 0) load_tree(f);
  while (f >= 0) {
    const int et = node_read<NW>(e, f);
    const bool fresh = is_new(f);  // starts as a lone root
    int cnt = fresh ? 1 : min(max(__builtin_amdgcn_readfirstlane(rec_cnt), 1), n_cap);
    const int cnt0 = fresh ? 0 : cnt;  // records below cnt0 stay as they are
    int ptok[Q], ppar[Q];  // parent -1: the root, or not a node
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int k = 64 * q + lane;
      ptok[q] = rec[q].x;
      ppar[q] = k < cnt && rec[q].y >= 0 && rec[q].y < k ? rec[q].y : -1;
      if (fresh && k == 0) ptok[q] = node_read<NW>(tok, f);
    }
    const int nf = pop_node<NW>(mine);
    if (nf >= 0) load_tree(nf);
    // every sub-tree whose root carries the token, in index order; its nodes in
    // index order too, so that a node's parent is mapped before the node
    int map[NW];  // draft node -> node of the pool tree (-1: dropped)
#pragma unroll
    for (int x = 0; x < NW; ++x) map[x] = -1;
    uint64_t roots[NW];
#pragma unroll
    for (int x = 0; x < NW; ++x) roots[x] = __ballot(live[x] && first[x] == f);
    for (int u; (u = pop_node<NW>(roots)) >= 0;) {
      uint64_t sub[NW];
#pragma unroll
      for (int x = 0; x < NW; ++x) {
        if (u == 64 * x + lane) map[x] = 0;
        const uint64_t a0 = anc[x][0], a1 = anc[x][NW - 1];
        sub[x] = __ballot(u != 64 * x + lane && (((u >= 64 ? a1 : a0) >> (u & 63)) & 1ull));
      }
      // The steps hang on each other only through map: a node's token and parent
      // are read by lane, its match in the tree is found by ballots, and all else
      // of a step is scalar.  Chains of 128 nodes (63 steps a tree on average),
      // 256 sequences: 143 us per call against 251 with the node and its
      // parent's image selected over both words and compared on three registers.
#pragma unroll
      for (int x = 0; x < NW; ++x)
        for (uint64_t m = sub[x]; m; m &= m - 1ull) {
          const int c = __builtin_ctzll(m);  // node 64 x + c
          const int pc = __builtin_amdgcn_readlane(par[x], c), tc = __builtin_amdgcn_readlane(tok[x], c);
          int pn = __builtin_amdgcn_readlane(map[0], pc & 63);
          if constexpr (NW == 2)
            if (x == 1) {  // (a node of the first word has its parent there)
              const int hi = __builtin_amdgcn_readlane(map[NW - 1], pc & 63);
              pn = pc >= 64 ? hi : pn;
            }
          int k = -1;  // full, or under a dropped node: skipped with its sub-tree
          if (pn >= 0) {
            uint64_t hit[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) hit[q] = __ballot(ppar[q] == pn) & __ballot(ptok[q] == tc);
#pragma unroll
            for (int q = Q - 1; q >= 0; --q) k = hit[q] ? 64 * q + __builtin_ctzll(hit[q]) : k;
            if (k < 0 && cnt < n_cap) {  // append as the last child of pn
              k = cnt++;
#pragma unroll
              for (int q = 0; q < Q; ++q)
                if (k == 64 * q + lane) {
                  ptok[q] = tc;
                  ppar[q] = pn;
                }
            }
          }
          map[x] = lane == c ? k : map[x];
        }
    }
    // a merge only appends
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int k = 64 * q + lane;
      if (k >= cnt0 && k < cnt) P.node[static_cast<size_t>(et) * n_cap + k] = make_int2(ptok[q], ppar[q]);
    }
    if (lane == 0) P.count[et] = cnt;
    f = nf;
  }

  if (__builtin_amdgcn_readfirstlane(arrived) != X - 1) return;
  // last to have read the table: token -> tree, slots claimed by compare-and-swap
#pragma unroll
  for (int x = 0; x < NW; ++x)
    if (newid[x] >= 0) {
      for (int s = home[x], k = 0; k < H; ++k, s = (s + 1) & (H - 1))
        if (atomicCAS(&P.tree[s], -1, newid[x]) == -1) {
          P.key[s] = tok[x];
          break;
        }
    }
  if (lane == 0) {
    *P.ntrees = min(ntrees0 + nnew, g.e_max);
    atomicExch(arrivals, 0);
  }
}

// One wave per sequence: node 64 q + lane of the tree in register q.  The root has
// depth 0; nodes that a pool not initialised leaves without a path to it are
// dropped.  Breadth first by levels as in stepping.  4.0 us for 16 trees of
// 65 nodes (5.5 with a thread per node and barriers): hash, count and node loads.
__global__ void __launch_bounds__(PTD_WAVE)
k_pool_retrieve(const void* pool, PoolGeom g, const int32_t* __restrict__ last_token,
                int T_max, int32_t* __restrict__ parent_out, int32_t* __restrict__ tokens_out,
                int32_t* __restrict__ tree_len_out) {
  constexpr int Q = kTreeRegs, N = Q * PTD_WAVE;
  __shared__ int s_dist[N], s_nxt[N], s_out[N], s_cnt[N];
  __shared__ uint64_t s_cm[N][Q];  // children
  const int lane = threadIdx.x, b = blockIdx.x;
  const PoolView P = view(const_cast<void*>(pool), g, b);
  int32_t* po = parent_out + static_cast<size_t>(b) * T_max;
  int32_t* to = tokens_out + static_cast<size_t>(b) * T_max;
#pragma unroll
  for (int q = 0; q < Q; ++q)
#pragma unroll
    for (int w = 0; w < Q; ++w) s_cm[64 * q + lane][w] = 0ull;
  // probe 64 slots at a time from the home slot
  const int key = last_token[b];
  int e = -1;
  const int home = home_slot(key, g.hbits);
  for (int k0 = 0; k0 < g.H; k0 += PTD_WAVE) {
    const int s = (home + k0 + lane) & (g.H - 1);
    const int tr = P.tree[s];
    const int ky = P.key[s];
    const uint64_t hit = __ballot(tr >= 0 && ky == key);
    const uint64_t empty = __ballot(tr < 0);
    const int fh = hit ? __builtin_ctzll(hit) : PTD_WAVE;
    const int fe = empty ? __builtin_ctzll(empty) : PTD_WAVE;
    if (fh < fe) {
      e = __builtin_amdgcn_readlane(tr, fh);
      if (e >= g.e_max) e = -1;  // out of range: a pool not initialised
      break;
    }
    if (fe < PTD_WAVE) break;  // an empty slot ends the probe: absent
  }
  int total = 0;
  if (e >= 0) {
    int2 nd[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int k = 64 * q + lane;
      nd[q] = k < g.n_cap ? P.node[static_cast<size_t>(e) * g.n_cap + k] : make_int2(0, -1);
    }
    const int cnt = min(max(P.count[e], 1), g.n_cap);
    // depth by pointer doubling; a chain that does not end at node 0 is marked
    int par[Q], dist[Q], nxt[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int k = 64 * q + lane;
      par[q] = k > 0 && k < cnt && nd[q].y >= 0 && nd[q].y < k ? nd[q].y : -1;
      dist[q] = par[q] >= 0 ? 1 : k == 0 ? 0 : kDeadNode;
      nxt[q] = par[q];
    }
    for (;;) {
      bool more = false;
#pragma unroll
      for (int q = 0; q < Q; ++q) more |= nxt[q] >= 0;
      if (!__any(more)) break;
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        s_dist[64 * q + lane] = dist[q];
        s_nxt[64 * q + lane] = nxt[q];
      }
      __syncthreads();  // (one wave: orders the LDS accesses)
#pragma unroll
      for (int q = 0; q < Q; ++q)
        if (nxt[q] >= 0) {
          dist[q] = min(dist[q] + s_dist[nxt[q]], kDeadNode);
          nxt[q] = s_nxt[nxt[q]];
        }
      __syncthreads();
    }
    bool reach[Q];
    int out[Q], pout[Q], sib[Q], nch[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      reach[q] = par[q] >= 0 && dist[q] < kDeadNode;
      total += __popcll(__ballot(reach[q]));
      if (reach[q]) atomicOr(reinterpret_cast<unsigned long long*>(&s_cm[par[q]][q]), 1ull << lane);
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      out[q] = pout[q] = -1;
      sib[q] = nch[q] = 0;
#pragma unroll
      for (int w = 0; w < Q; ++w) {
        const uint64_t sm = s_cm[max(par[q], 0)][w];
        sib[q] += w < q ? __popcll(sm) : w == q ? __popcll(sm & below_mask(lane)) : 0;
        nch[q] += __popcll(s_cm[64 * q + lane][w]);
      }
      if (reach[q] && dist[q] == 1) {  // the root's children, in insertion order
        out[q] = sib[q];
        s_out[64 * q + lane] = out[q];
      }
    }
    int lo = 0, hi = __builtin_amdgcn_readlane(nch[0], 0);
    for (int L = 1; hi < total; ++L) {  // uniform; every level has children up to the last
      const int len = hi - lo;
#pragma unroll
      for (int q = 0; q < Q; ++q)
        if (reach[q] && dist[q] == L) s_cnt[out[q] - lo] = nch[q];
      __syncthreads();
      int run = hi;
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const int pos = 64 * q + lane;
        int sum;
        const int x = wave_excl_sum(pos < len ? s_cnt[pos] : 0, &sum);
        if (pos < len) s_cnt[pos] = run + x;
        run += sum;
      }
      __syncthreads();
#pragma unroll
      for (int q = 0; q < Q; ++q)
        if (reach[q] && dist[q] == L + 1) {
          pout[q] = s_out[par[q]];
          out[q] = s_cnt[pout[q] - lo] + sib[q];
          s_out[64 * q + lane] = out[q];
        }
      lo = hi;
      hi = run;
      __syncthreads();
    }
#pragma unroll
    for (int q = 0; q < Q; ++q)
      if (reach[q] && out[q] < T_max) {
        po[out[q]] = pout[q];
        to[out[q]] = nd[q].x;
      }
  }
  for (int t = total + lane; t < T_max; t += PTD_WAVE) {
    po[t] = -1;
    to[t] = -1;
  }
  if (lane == 0) tree_len_out[b] = min(total, T_max);
}

}  // namespace

extern "C" size_t ptd_pool_bytes(int32_t B, int32_t e_max, int32_t n_cap) {
  PoolGeom g;
  if (B < 1 || !pool_geom(e_max, n_cap, &g)) return 0;
  return static_cast<size_t>(B) * g.seq_bytes;
}

extern "C" int ptd_pool_init(void* pool, size_t pool_bytes, int32_t B, int32_t e_max,
                             int32_t n_cap, void* stream) {
  PTD_RETURN_IF(!pool, PTD_ERR_NULL);
  PoolGeom g;
  PTD_RETURN_IF(B < 1 || !pool_geom(e_max, n_cap, &g), PTD_ERR_SHAPE);
  PTD_RETURN_IF(pool_bytes < static_cast<size_t>(B) * g.seq_bytes, PTD_ERR_WORKSPACE);
  PTD_RETURN_IF(!ptd_aligned(pool, 256), PTD_ERR_ALIGN);
  hipLaunchKernelGGL(k_pool_init, dim3(B), dim3(kInitThreads), 0,
                     static_cast<hipStream_t>(stream), pool, g);
  return ptd_launch_status();
}

extern "C" int ptd_pool_merge(void* pool, size_t pool_bytes, int32_t B, int32_t e_max,
                              int32_t n_cap, const int32_t* parent, const int32_t* tokens,
                              const int32_t* tree_len, int32_t T, int32_t* dev_status,
                              void* stream) {
  PTD_RETURN_IF(!pool || !parent || !tokens, PTD_ERR_NULL);
  PoolGeom g;
  PTD_RETURN_IF(B < 1 || !pool_geom(e_max, n_cap, &g) || T < 1 || T > kMaxNodes, PTD_ERR_SHAPE);
  PTD_RETURN_IF(pool_bytes < static_cast<size_t>(B) * g.seq_bytes, PTD_ERR_WORKSPACE);
  PTD_RETURN_IF(!ptd_aligned(pool, 256), PTD_ERR_ALIGN);
  // Two touched trees per wave at most, four where the waves' repeated look-ups
  // add up (us per call of 64 nodes, two / four: B = 16 10.3 / 11.7, 128 12.0 /
  // 12.7, 256 19.2 / 14.7; 96 nodes, B = 64 18.5 / 20.8, 128 24.0 / 20.3).  At most
  // 2^32 threads.
  const int per_wave = static_cast<long long>(B) * T <= 8192 ? 2 : 4;
  const int X = std::max(1, std::min(ptd_cdiv(T, per_wave), (1 << 25) / B));
  const dim3 grid(static_cast<unsigned>(B) * X);
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int nw = T <= PTD_WAVE ? 1 : 2, q = ptd_cdiv(n_cap, PTD_WAVE);
#define PTD_MERGE(nw_, q_)                                                                      \
  if (nw == nw_ && q == q_)                                                                     \
    hipLaunchKernelGGL((k_pool_merge<nw_, q_>), grid, dim3(PTD_WAVE), 0, st, pool, g, parent,   \
                       tokens, tree_len, T, X, dev_status);
  PTD_MERGE(1, 1) PTD_MERGE(1, 2) PTD_MERGE(1, 3) PTD_MERGE(2, 1) PTD_MERGE(2, 2) PTD_MERGE(2, 3)
#undef PTD_MERGE
  return ptd_launch_status();
}

extern "C" int ptd_pool_retrieve(const void* pool, size_t pool_bytes, int32_t B, int32_t e_max,
                                 int32_t n_cap, const int32_t* last_token, int32_t T_max,
                                 int32_t* parent_out, int32_t* tokens_out,
                                 int32_t* tree_len_out, void* stream) {
  PTD_RETURN_IF(!pool || !last_token || !parent_out || !tokens_out || !tree_len_out,
                PTD_ERR_NULL);
  PoolGeom g;
  PTD_RETURN_IF(B < 1 || !pool_geom(e_max, n_cap, &g) || T_max < 1 || T_max > PTD_MAX_T,
                PTD_ERR_SHAPE);
  PTD_RETURN_IF(pool_bytes < static_cast<size_t>(B) * g.seq_bytes, PTD_ERR_WORKSPACE);
  PTD_RETURN_IF(!ptd_aligned(pool, 256), PTD_ERR_ALIGN);
  hipLaunchKernelGGL(k_pool_retrieve, dim3(B), dim3(PTD_WAVE), 0,
                     static_cast<hipStream_t>(stream), pool, g, last_token, T_max, parent_out,
                     tokens_out, tree_len_out);
  return ptd_launch_status();
}

extern "C" int ptd_step_prune(const int32_t* parent, const int32_t* tokens,
                              const int32_t* tree_len, int32_t B, int32_t T, int32_t d_max,
                              int32_t T_max, int32_t* parent_next, int32_t* tokens_next,
                              int32_t* tree_len_next, int32_t* dev_status, void* stream) {
  PTD_RETURN_IF(!parent || !tokens || !parent_next || !tokens_next || !tree_len_next,
                PTD_ERR_NULL);
  PTD_RETURN_IF(B < 1 || T < 1 || T > kMaxNodes || d_max < 1 || T_max < 1 ||
                    T_max > PTD_MAX_T,
                PTD_ERR_SHAPE);
  if (T <= PTD_WAVE)
    hipLaunchKernelGGL(k_step_prune<1>, dim3(B), dim3(PTD_WAVE), 0,
                       static_cast<hipStream_t>(stream), parent, tokens, tree_len, T, d_max, T_max,
                       parent_next, tokens_next, tree_len_next, dev_status);
  else
    hipLaunchKernelGGL(k_step_prune<2>, dim3(B), dim3(PTD_WAVE), 0,
                       static_cast<hipStream_t>(stream), parent, tokens, tree_len, T, d_max, T_max,
                       parent_next, tokens_next, tree_len_next, dev_status);
  return ptd_launch_status();
}
