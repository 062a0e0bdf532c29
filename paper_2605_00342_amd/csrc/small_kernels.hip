// Integer / latency-bound parts of the verification step: EVICT prefix selection
// (Sec. 3.1-3.2), greedy acceptance (Sec. 2.1, temperature 0), the expert union and the
// token grouping it induces (Eq. 5), row gather for tree compaction.
#include <stdarg.h>
#include <string.h>

#include <mutex>

#include "ctx.h"
#include "union_device.h"

namespace evict {

static thread_local char g_err[512] = "";

void set_error(const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
}

namespace {

constexpr int kSelThreads = 1024;       // one tree of more than 64 nodes
constexpr int kSelThreadsSmall = 256;   // batches of trees of at most 64 nodes on average: mostly one wavefront's work
constexpr int kMaxSel = EVICT_MAX_SELECT_NODES;

// Kept-set compaction of one tree: nodes with rank < kstar, ascending node id; parents
// re-indexed into the kept set. s_flag/s_new are LDS arrays of n ints.
__device__ void compact_tree(int n, int kstar, const int* s_par, const int* s_rank, int* s_new, int* s_wave,
                             int32_t* keep_out, int32_t* newpar_out) {
  const int tid = threadIdx.x;
  // 4 consecutive nodes per thread so that the scan keeps node order
  int f[4], cnt = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    int i = tid * 4 + j;
    f[j] = (i < n && s_rank[i] < kstar) ? 1 : 0;
    cnt += f[j];
  }
  int total;
  int base = block_excl_scan(cnt, s_wave, &total);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    int i = tid * 4 + j;
    if (i < n) s_new[i] = f[j] ? base : -1;
    base += f[j];
  }
  __syncthreads();
  for (int i = tid; i < n; i += blockDim.x) {
    int ni = s_new[i];
    if (ni >= 0) {
      keep_out[ni] = i;
      int p = s_par[i];
      newpar_out[ni] = p < 0 ? -1 : s_new[p];
    }
  }
}

// One tree of at most 64 nodes in one wavefront, node i in lane i, everything in registers and
// cross-lane operations: the same arithmetic in the same order as the workgroup path of select_prefix_kernel (one
// rounded multiply per node top-down, ranking by (score descending, index ascending), sequential
// fp32 running sum, IEEE division, first maximum), without LDS round trips and barriers.
// Arrays start at the tree's first node. Every lane returns its rank, its (checked) parent, k* and S_{k*}.
struct WaveSelection { int rank, parent, kstar; float est; };
__device__ __forceinline__ WaveSelection select_wave(
    const int32_t* __restrict__ parent, const float* __restrict__ prob, const float* __restrict__ cost, int kmax, int n,
    float rho, int32_t* __restrict__ order_out, float* __restrict__ psum_out, int32_t* __restrict__ status) {
  const int lane = lane_id();
  const bool live = lane < n;
  int p = -1;
  float q = 0.0f, c = 1.0f;
  if (live) {
    int bad_in = 0;
    p = parent[lane];
    q = prob[lane];
    if (cost && lane < kmax) c = cost[lane + 1];  // C(lane + 1)
    if (lane == 0) p = -1;
    else if (p < 0 || p >= lane) { p = 0; bad_in |= ST_BAD_PARENT; }  // invalid ids are clamped and flagged
    // a probability outside [0, 1] (or NaN) could rank a child above its parent and break the ancestor-closure
    // of the prefixes (Sec. 3.2.1): clamped and flagged; an unusable cost entry is never selected
    if (lane > 0 && !(q >= 0.0f && q <= 1.0f)) { q = q > 1.0f ? 1.0f : 0.0f; bad_in |= ST_BAD_PROB; }
    if (!(c > 0.0f)) { c = 0.0f; bad_in |= ST_BAD_COST; }
    if (bad_in && status) atomicOr(status, bad_in);
  }
  // depth by walking up in lock step
  int dep = 0, a = p;
  while (__ballot(a >= 0)) {
    const int up = __shfl(p, a < 0 ? 0 : a);
    if (a >= 0) { ++dep; a = up; }
  }
  int maxdep = dep;
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    const int other = __shfl_xor(maxdep, o);
    maxdep = other > maxdep ? other : maxdep;
  }
  // Score(v) = Score(parent(v)) * q(v), level by level (Eq. 7); the root counts as probability 1
  float sc = lane == 0 ? 1.0f : 0.0f;
  for (int lvl = 1; lvl <= maxdep; ++lvl) {
    const float sp = __shfl(sc, p < 0 ? 0 : p);
    if (live && dep == lvl) sc = __fmul_rn(sp, q);
  }
  // rank by (score descending, index ascending); lanes past the tree keep their own position
  int r = 0;
  const int sbits = __float_as_int(sc);
  for (int j0 = 0; j0 < n; j0 += 8) {  // (lanes past the tree hold zeros and come after every node: never counted)
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float sj = __int_as_float(__builtin_amdgcn_readlane(sbits, j0 + j));
      r += (sj > sc || (sj == sc && j0 + j < lane)) ? 1 : 0;
    }
  }
  r = live ? r : lane;
  if (live && order_out) order_out[r] = lane;
  // scores in rank order: lane i sends its score to lane r
  const int sorted_bits = __builtin_amdgcn_ds_permute(r << 2, live ? sbits : 0);
  // S_k: sequential fp32 running sum over the ranking
  float acc = 0.0f, S = 0.0f;
  for (int j0 = 0; j0 < n; j0 += 8) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      acc = __fadd_rn(acc, __int_as_float(__builtin_amdgcn_readlane(sorted_bits, j0 + j)));
      if (lane == j0 + j) S = acc;
    }
  }
  if (live && psum_out) psum_out[lane] = S;
  const int kk = n < kmax ? n : kmax;
  const float total = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(S), n - 1));
  float bv = -1.0f;
  int bi = 0x7fffffff;
  if (lane < kk) {
    bv = rho >= 0.0f ? (__fdiv_rn(S, total) >= rho ? 1.0f : 0.0f) : (c > 0.0f ? __fdiv_rn(S, c) : -1.0f);
    bi = lane;
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    const float ov = __shfl_xor(bv, o);
    const int oi = __shfl_xor(bi, o);
    if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
  }
  if (rho >= 0.0f && bv == 0.0f) bi = kk - 1;  // coverage not reached within kmax: the whole budget
  const int kstar = bi + 1;
  const float est = __shfl(S, bi);
  return WaveSelection{r, p, kstar, est};
}

// how many of the four scores s4 of nodes j .. j + 3 rank before node i of score si (LDS broadcast reads, four at a time)
__device__ __forceinline__ int rank_among4(const float4 s4, int j, float si, int i) {
  int r = (s4.x > si || (s4.x == si && j < i)) ? 1 : 0;
  r += (s4.y > si || (s4.y == si && j + 1 < i)) ? 1 : 0;
  r += (s4.z > si || (s4.z == si && j + 2 < i)) ? 1 : 0;
  r += (s4.w > si || (s4.w == si && j + 3 < i)) ? 1 : 0;
  return r;
}

// One workgroup per tree. Writes k*, S_{k*}, the ranking and the running sums; when
// `single` it also writes the compacted tree (B == 1), otherwise ranks go to rank_ws for
// the second kernel.
__global__ __launch_bounds__(kSelThreads) void select_prefix_kernel(
    const int32_t* __restrict__ tree_off, const int32_t* __restrict__ parent, const float* __restrict__ prob,
    const float* __restrict__ cost, int kmax, int32_t* __restrict__ k_star, float* __restrict__ est_len,
    int32_t* __restrict__ order_out, float* __restrict__ psum_out, int32_t* rank_ws, int single, int32_t* keep,
    int32_t* new_parent, int32_t* __restrict__ new_tree_off, int n_single, float rho, int32_t* __restrict__ status) {
  __shared__ int s_par[kMaxSel];
  __shared__ __attribute__((aligned(16))) float s_score[kMaxSel];
  __shared__ float s_sorted[kMaxSel];
  __shared__ float s_prob[kMaxSel];
  __shared__ float s_cost[kMaxSel];
  __shared__ int s_rank[kMaxSel];
  __shared__ int s_aux[kMaxSel];  // depth, later new index
  __shared__ int s_wave[16];
  __shared__ float s_bestv[16];
  __shared__ int s_besti[16];
  __shared__ int s_maxdep;

  const int b = blockIdx.x, tid = threadIdx.x, lane = lane_id(), w = tid >> 6;
  const int nthreads = blockDim.x, nwaves = nthreads >> 6;
  // a single tree spans [0, T): its offsets need not be fetched
  const int lo = n_single > 0 ? 0 : tree_off[b];
  int n = n_single > 0 ? n_single : tree_off[b + 1] - lo;
  n = n < 1 ? 1 : (n > kMaxSel ? kMaxSel : n);
  if (!single && n <= 64) {
    // a small tree of a batch fits one wavefront's registers: 12 -> 8 us for trees of 64 nodes
    if (w > 0) return;  // (whole wavefronts, before any barrier)
    const WaveSelection sel = select_wave(parent + lo, prob + lo, cost, kmax, n, rho, order_out ? order_out + lo : nullptr,
                                          psum_out ? psum_out + lo : nullptr, status);
    if (lane < n) rank_ws[lo + lane] = sel.rank;
    if (lane == 0) {
      k_star[b] = sel.kstar;
      est_len[b] = sel.est;
    }
    return;
  }

  if (tid == 0) s_maxdep = 0;
  int bad_in = 0;
  for (int i = tid; i < n; i += nthreads) {
    int p = parent[lo + i];
    if (i == 0) p = -1;
    else if (p < 0 || p >= i) { p = 0; bad_in |= ST_BAD_PARENT; }  // invalid ids are clamped and flagged
    s_par[i] = p;
    // all global reads issued together, up front. A probability outside [0, 1] (or NaN) could rank a child
    // above its parent and break the ancestor-closure of the prefixes (Sec. 3.2.1): it is clamped and flagged.
    float q = prob[lo + i];
    if (i > 0 && !(q >= 0.0f && q <= 1.0f)) { q = q > 1.0f ? 1.0f : 0.0f; bad_in |= ST_BAD_PROB; }
    s_prob[i] = q;
    float c = (cost && i < kmax) ? cost[i + 1] : 1.0f;  // s_cost[i] = C(i + 1)
    if (!(c > 0.0f)) { c = 0.0f; bad_in |= ST_BAD_COST; }  // (never selected below)
    s_cost[i] = c;
    s_rank[i] = 0;
  }
  if (bad_in && status) atomicOr(status, bad_in);
  __syncthreads();
  // depth of every node (walk to the root; parent ids strictly decrease)
  int mydep_max = 0;
  for (int i = tid; i < n; i += nthreads) {
    int dep = 0;
    for (int p = s_par[i]; p >= 0; p = s_par[p]) ++dep;
    s_aux[i] = dep;
    mydep_max = dep > mydep_max ? dep : mydep_max;
  }
  atomicMax(&s_maxdep, mydep_max);
  if (tid == 0) s_score[0] = 1.0f;  // the root counts as probability 1 (Eq. 7)
  __syncthreads();
  const int maxdep = s_maxdep;
  // Score(v) = Score(parent(v)) * q(v): one rounded fp32 multiply per node, level by level
  for (int lvl = 1; lvl <= maxdep; ++lvl) {
    for (int i = tid; i < n; i += nthreads)
      if (s_aux[i] == lvl) s_score[i] = __fmul_rn(s_score[s_par[i]], s_prob[i]);
    __syncthreads();
  }
  // rank by (score descending, index ascending): the scores a node is compared with are shared out among `parts` threads
  // per node, so that all threads have work whatever the size of the tree (400 nodes: 46 us with one of 256 threads per
  // node, 21 us this way; 32 such trees)
  const int npad = (n + 63) & ~63;
  const int parts = nthreads >= 2 * npad ? nthreads / npad : 1;
  if (parts > 1) {
    const int part = tid / npad, i = tid - part * npad;
    const int per = ((n + parts - 1) / parts + 3) & ~3;
    if (part < parts && i < n) {
      const float si = s_score[i];
      int r = 0;
      const int j1 = (part + 1) * per < n ? (part + 1) * per : n;
      int j = part * per;
#pragma unroll 2
      for (; j + 4 <= j1; j += 4) r += rank_among4(*reinterpret_cast<const float4*>(&s_score[j]), j, si, i);
      for (; j < j1; ++j) r += (s_score[j] > si || (s_score[j] == si && j < i)) ? 1 : 0;
      atomicAdd(&s_rank[i], r);
    }
    __syncthreads();
    for (int i2 = tid; i2 < n; i2 += nthreads) {
      const int r = s_rank[i2];
      s_sorted[r] = s_score[i2];
      if (order_out) order_out[lo + r] = i2;
    }
  } else {
    for (int i = tid; i < n; i += nthreads) {
      const float si = s_score[i];
      int r = 0;
      int j = 0;
#pragma unroll 2
      for (; j + 4 <= n; j += 4) r += rank_among4(*reinterpret_cast<const float4*>(&s_score[j]), j, si, i);
      for (; j < n; ++j) r += (s_score[j] > si || (s_score[j] == si && j < i)) ? 1 : 0;
      s_rank[i] = r;
      s_sorted[r] = si;
      if (order_out) order_out[lo + r] = i;
    }
  }
  __syncthreads();
  // S_k: sequential fp32 running sum over the ranking (one wavefront, lane broadcast)
  if (w == 0) {
    float acc = 0.0f;
    for (int c = 0; c < n; c += 64) {
      const int idx = c + lane;
      const int vbits = __float_as_int(idx < n ? s_sorted[idx] : 0.0f);
      float mine = 0.0f;
      const int lim = (n - c) < 64 ? (n - c) : 64;
      for (int j0 = 0; j0 < lim; j0 += 8) {  // (lanes past the tree hold zeros)
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          acc = __fadd_rn(acc, __int_as_float(__builtin_amdgcn_readlane(vbits, j0 + j)));
          if (lane == j0 + j) mine = acc;
        }
      }
      if (idx < n) s_sorted[idx] = mine;  // now holds S_{idx+1}
    }
  }
  __syncthreads();
  // u_k = S_k / cost[k]; k* = smallest k attaining the maximum over 1..min(n, kmax)
  const int kk = n < kmax ? n : kmax;
  float bv = -1.0f;
  int bi = 0x7fffffff;
  for (int i = tid; i < n; i += nthreads) {
    const float S = s_sorted[i];
    if (psum_out) psum_out[lo + i] = S;
    if (i < kk) {
      // cost-aware rule: u_k = S_k / C(k). Coverage rule (rho >= 0, the cost-agnostic ablation of
      // Sec. 4.3.2): u_k = 1 where S_k / S_n >= rho, else 0, so that the first maximum is the
      // smallest prefix reaching the coverage.
      float u;
      if (rho >= 0.0f) u = __fdiv_rn(S, s_sorted[n - 1]) >= rho ? 1.0f : 0.0f;
      else u = s_cost[i] > 0.0f ? __fdiv_rn(S, s_cost[i]) : -1.0f;  // (a flagged, unusable cost entry is never the maximum)
      if (u > bv || (u == bv && i < bi)) { bv = u; bi = i; }
    }
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    const float ov = __shfl_xor(bv, o);
    const int oi = __shfl_xor(bi, o);
    if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
  }
  if (lane == 0) { s_bestv[w] = bv; s_besti[w] = bi; }
  __syncthreads();
  bv = s_bestv[0]; bi = s_besti[0];
  for (int i = 1; i < nwaves; ++i) {
    const float ov = s_bestv[i];
    const int oi = s_besti[i];
    if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
  }
  if (rho >= 0.0f && bv == 0.0f) bi = kk - 1;  // coverage not reached within kmax: the whole budget
  const int kstar = bi + 1;
  if (tid == 0) {
    k_star[b] = kstar;
    est_len[b] = s_sorted[bi];
  }
  if (single) {
    if (tid == 0) { new_tree_off[0] = 0; new_tree_off[1] = kstar; }
    compact_tree(n, kstar, s_par, s_rank, s_aux, s_wave, keep, new_parent);
  } else {
    for (int i = tid; i < n; i += nthreads) rank_ws[lo + i] = s_rank[i];
  }
}

// a single tree of at most 64 nodes: selection and compaction in one wavefront
__global__ __launch_bounds__(64) void select_prefix_wave_kernel(
    const int32_t* __restrict__ parent, const float* __restrict__ prob, const float* __restrict__ cost, int kmax, int n,
    float rho, int32_t* __restrict__ k_star, float* __restrict__ est_len, int32_t* __restrict__ order_out,
    float* __restrict__ psum_out, int32_t* __restrict__ keep, int32_t* __restrict__ new_parent,
    int32_t* __restrict__ new_tree_off, int32_t* __restrict__ status) {
  const int lane = threadIdx.x;
  const bool live = lane < n;
  const WaveSelection sel = select_wave(parent, prob, cost, kmax, n, rho, order_out, psum_out, status);
  const int r = sel.rank, p = sel.parent, kstar = sel.kstar;
  // kept nodes ascending, parents re-indexed by counting kept nodes below
  const unsigned long long kept = __ballot(live && r < kstar);
  if (live && r < kstar) {
    const int ni = __popcll(kept & ((1ull << lane) - 1ull));
    keep[ni] = lane;
    new_parent[ni] = p < 0 ? -1 : __popcll(kept & ((1ull << p) - 1ull));
  }
  if (lane == 0) {
    k_star[0] = kstar;
    est_len[0] = sel.est;
    new_tree_off[0] = 0;
    new_tree_off[1] = kstar;
  }
}

// Second step for batches: one workgroup compacts all trees, one wavefront per tree. Tree b's compacted output starts at
// or before tree b's own input offset and so lands on the ranks of earlier trees (rank_ws aliases new_parent): the ranks
// of a group of trees are taken into LDS, with the parents, before any of its output is written, and a group is as many
// trees as fit there (kCompactNodes nodes, one tree per thread in the scans). 16 trees of 64 nodes: 20 us with the trees
// walked one after the other by the whole workgroup, 4 us this way.
constexpr int kCompactThreads = 1024;
constexpr int kCompactNodes = 10 * 1024;
static_assert(kCompactNodes >= kMaxSel && kMaxSel <= 0xFFFF, "a tree fits a group; ranks and ids fit 16 bits");
__global__ __launch_bounds__(kCompactThreads) void compact_batch_kernel(
    const int32_t* __restrict__ tree_off, const int32_t* __restrict__ parent, const int32_t* __restrict__ k_star,
    int B, int32_t* rank_ws, int32_t* keep, int32_t* new_parent, int32_t* __restrict__ new_tree_off) {
  __shared__ uint32_t s_node[kCompactNodes];  // parent << 16 (0xFFFF: root) | rank, later the new id
  __shared__ int s_lo[kCompactThreads], s_n[kCompactThreads], s_ks[kCompactThreads], s_at[kCompactThreads], s_out[kCompactThreads];
  __shared__ int s_wave[16];
  const int tid = threadIdx.x, lane = lane_id();
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  int out = 0;
  for (int b0 = 0; b0 < B;) {
    // this thread's tree, where its nodes sit in LDS and its output, and how many trees the group holds
    const int b = b0 + tid;
    int lo = 0, n = 0, ks = 0;
    if (b < B) {
      lo = tree_off[b];
      n = tree_off[b + 1] - lo;
      n = n < 1 ? 1 : (n > kMaxSel ? kMaxSel : n);
      ks = k_star[b];
    }
    int total;
    const int at = block_excl_scan(n, s_wave, &total);
    const bool in = b < B && at + n <= kCompactNodes;
    const int ntrees = __syncthreads_count(in);
    const int before = block_excl_scan(in ? ks : 0, s_wave, &total);
    if (in) {
      s_lo[tid] = lo; s_n[tid] = n; s_ks[tid] = ks; s_at[tid] = at;
      s_out[tid] = out + before;
      new_tree_off[b] = out + before;
    }
    __syncthreads();
    for (int t = w; t < ntrees; t += kCompactThreads / 64) {
      const int tlo = s_lo[t], tn = s_n[t], tat = s_at[t];
      for (int i = lane; i < tn; i += 64) {
        int p = parent[tlo + i];
        if (i == 0) p = 0xFFFF;
        else if (p < 0 || p >= i) p = 0;
        s_node[tat + i] = ((uint32_t)p << 16) | (uint32_t)rank_ws[tlo + i];
      }
    }
    __syncthreads();  // every rank of the group is in LDS before its first output is written
    for (int t = w; t < ntrees; t += kCompactThreads / 64) {
      const int tn = s_n[t], tks = s_ks[t], tout = s_out[t];
      uint32_t* node = s_node + s_at[t];
      int kept = 0;
      for (int c0 = 0; c0 < tn; c0 += 64) {  // nodes in ascending order: a parent has its new id before its children ask
        const int i = c0 + lane;
        const uint32_t v = i < tn ? node[i] : 0xFFFFu;
        const bool keeps = i < tn && (int)(v & 0xFFFFu) < tks;
        const unsigned long long m = __ballot(keeps);
        const int ni = kept + __popcll(m & ((1ull << lane) - 1ull));
        if (keeps) node[i] = (v & 0xFFFF0000u) | (uint32_t)ni;
        wave_lds_fence();
        if (keeps) {
          const uint32_t p = v >> 16;
          keep[tout + ni] = i;
          new_parent[tout + ni] = p == 0xFFFFu ? -1 : (int)(node[p] & 0xFFFFu);
        }
        kept += __popcll(m);
      }
    }
    out += total;
    b0 += ntrees;
    __syncthreads();
  }
  if (tid == 0) new_tree_off[B] = out;
}

// One wavefront per tree; the tree is staged in LDS so the walk has no global-memory latency.
__global__ __launch_bounds__(64) void accept_path_kernel(
    const int32_t* __restrict__ tree_off, const int32_t* __restrict__ parent, const int32_t* __restrict__ tok,
    const int32_t* __restrict__ next, int32_t* __restrict__ path, int path_stride, int32_t* __restrict__ path_len,
    int32_t* __restrict__ bonus) {
  __shared__ int s_par[kMaxSel];
  __shared__ int s_tok[kMaxSel];
  __shared__ int s_next[kMaxSel];
  const int b = blockIdx.x, lane = threadIdx.x;
  const int lo = tree_off[b];
  int n = tree_off[b + 1] - lo;
  n = n < 1 ? 1 : (n > kMaxSel ? kMaxSel : n);
  for (int i = lane; i < n; i += 64) {
    s_par[i] = parent[lo + i];
    s_tok[i] = tok[lo + i];
    s_next[i] = next[lo + i];
  }
  int32_t* my = path + (size_t)b * path_stride;
  for (int i = lane; i < path_stride; i += 64) my[i] = i == 0 ? 0 : -1;
  __syncthreads();
  int cur = 0, len = 1;
  while (true) {
    const int want = s_next[cur];
    int found = -1;
    for (int base = cur + 1; base < n; base += 64) {
      const int c = base + lane;
      const bool m = c < n && s_par[c] == cur && s_tok[c] == want;
      const unsigned long long mask = __ballot(m);
      if (mask) { found = base + __ffsll((long long)mask) - 1; break; }
    }
    if (found < 0) break;
    cur = found;  // strictly increasing: the walk ends
    if (lane == 0 && len < path_stride) my[len] = cur;
    ++len;
  }
  if (lane == 0) { path_len[b] = len; bonus[b] = s_next[cur]; }
}

// ------------------------------------------------------------------------------------
// Acceptance under sampling: the sequential sibling rule (Sec. 2.1, Eq. 3).
// ------------------------------------------------------------------------------------
constexpr int kSampThreads = 1024;
constexpr int kSampWaves = kSampThreads / 64;
// Floats of scratch per node: the maxima of kSampWaves parts of the row, then their sums of exponentials. Behind those of node b
// lies what the walk of tree b hands to its draw: the kSampWaves segment sums, the segments' maxima that they are relative to, and
// the last node of the walk (bits of an int). (By the tree's number, not at its root: an empty tree's offset is the next tree's root, or past the end.)
constexpr int kSampStats = EVICT_SAMP_STATS;
constexpr int kSampSeg = 2 * kSampWaves, kSampSegMax = 3 * kSampWaves, kSampCur = 4 * kSampWaves;
static_assert(kSampStats > kSampCur, "maxima, sums; segment sums, their maxima, last node");

// Per node, what turns any logit of the row into a probability: for each of kSampWaves contiguous parts of the vocabulary its maximum
// and its sum of exp((logit - that maximum) / temperature), one wavefront per (row, part), so that a few rows still fill the
// chip: a row is 0.6 MB at a vocabulary of 151936, and one workgroup walking it alone is bound by the latency of its loads.
// One pass: every lane keeps the maximum of what it has seen and rescales its sum when that grows; the sums of rows of 151936 drawn
// with deviations of 1 to 5 are off from those in 64 bits by 1.05e-7 relative in the mean, 4.4e-7 at most (with the row's maximum found
// first, in a pass of its own, 1.25e-7 and 9.4e-7). `skip_leaves`: a node without children needs neither number, as the walk ends
// there, and the draw takes maxima and sums of its own; that is about half of the nodes of a tree. (113 rows of 151936, us: two passes
// over all rows 12.2 + 13.5, this way 11.3, about 38 MB; what is left is the launch, two trips for the tree and the parents, and one
// workgroup per CU of loads.) The order of every addition is fixed by the vocabulary size alone.
constexpr int kStatsThreads = 256;
constexpr int kStatsWgs = kSampThreads / kStatsThreads;  // workgroups per row
constexpr int kStatsBatch = 32;                          // loads in flight per lane

// exp((v - m) / temperature), zero while nothing but -inf has been seen
__device__ __forceinline__ float samp_exp(float v, float m, float inv_temp) { return __expf((v - (m == -INFINITY ? 0.0f : m)) * inv_temp); }

__global__ __launch_bounds__(kStatsThreads) void row_stats_kernel(const float* __restrict__ logits, int V, float inv_temp, float* __restrict__ stats,
                                                                  int T, const int* __restrict__ t_dev, const int32_t* __restrict__ tree_off,
                                                                  const int32_t* __restrict__ parent, int B, int skip_leaves) {
  const int r = (int)blockIdx.x / kStatsWgs;
  if (r >= dyn_tokens(t_dev, T)) return;  // (rows past the call's actual token count)
  const int lane = threadIdx.x & 63;
  if (skip_leaves) {
    // the tree of row r: the first that ends past it
    int b = 0;
    for (; b < B; b += 64) {
      const unsigned long long past = __ballot(b + lane < B && tree_off[b + lane + 1] > r);
      if (past) { b += __ffsll((long long)past) - 1; break; }
    }
    if (b < B) {
      const int lo = tree_off[b], node = r - lo;
      int end = tree_off[b + 1];
      end = end < T ? end : T;
      bool parent_of = node <= 0;  // (the root also takes nodes whose parent is invalid)
      for (int c0 = r + 1; c0 < end && !parent_of; c0 += 64) parent_of = __ballot(c0 + lane < end && parent[c0 + lane] == node) != 0;
      if (!parent_of) return;
    }
  }
  const int part = ((int)blockIdx.x % kStatsWgs) * (kStatsThreads / 64) + (threadIdx.x >> 6);
  const float* row = logits + (size_t)r * V;
  const int seg = (V + kSampWaves - 1) / kSampWaves;
  const int lo = part * seg, hi = lo + seg < V ? lo + seg : V;
  float m = -INFINITY, z = 0.0f;
  float v[2][kStatsBatch];  // one batch is on its way while the other is added up
  auto request = [&](float(&to)[kStatsBatch], int i0) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < kStatsBatch; ++u) {
      const int i = i0 + u * 64 + lane;
      to[u] = i < hi ? row[i] : -INFINITY;
    }
  };
  auto add = [&](const float(&of)[kStatsBatch]) __attribute__((always_inline)) {
    float top = m;
#pragma unroll
    for (int u = 0; u < kStatsBatch; ++u) top = fmaxf(top, of[u]);
    z *= samp_exp(m, top, inv_temp);
    m = top;
#pragma unroll
    for (int u = 0; u < kStatsBatch; ++u) z += samp_exp(of[u], m, inv_temp);
  };
  constexpr int kStep = 64 * kStatsBatch;
  request(v[0], lo);
  for (int i0 = lo; i0 < hi; i0 += 2 * kStep) {
    if (i0 + kStep < hi) request(v[1], i0 + kStep);
    add(v[0]);
    if (i0 + kStep >= hi) break;
    if (i0 + 2 * kStep < hi) request(v[0], i0 + 2 * kStep);
    add(v[1]);
  }
  const float top = wave_max(m);
  z = wave_sum(z * samp_exp(m, top, inv_temp));
  if (lane == 0) {
    stats[(size_t)r * kSampStats + part] = top;
    stats[(size_t)r * kSampStats + kSampWaves + part] = z;
  }
}

// maximum of a row from those of its parts
__device__ __forceinline__ float stats_max(const float* __restrict__ st) {
  float m = -INFINITY;
#pragma unroll
  for (int i = 0; i < kSampWaves; ++i) m = fmaxf(m, st[i]);
  return m;
}
// its sum, relative to that maximum
__device__ __forceinline__ float stats_sum(const float* __restrict__ st, float m, float inv_temp) {
  float z = 0.0f;
#pragma unroll
  for (int i = 0; i < kSampWaves; ++i) z += st[kSampWaves + i] * samp_exp(st[i], m, inv_temp);
  return z;
}

// Short rows: both numbers by one workgroup per row, the maximum of the whole row first, then the sum relative to it; they go side by side to the
// first two slots, as the walk fetches them for every node's parent (1024 nodes of 16384 logits, all launches, us: 42.6, and 44.2 with the
// sum 64 bytes behind the maximum). In parts, by the kernel above, the same takes (trees of 32 nodes, four of 32, eight of 64) 16.6, 17.1, 20.3 at 4000
// logits, here 12.4, 12.8, 14.9; at 8000 15.9, 16.6, 20.8 (13.9, 14.3, 18.0), at 12000 16.3, 17.4, 21.6 (15.8, 18.1, 22.9). At 16384 the parts are the
// faster, 16.8, 17.7, 22.5 (18.4, 20.7, 25.5): the line was drawn when they took a launch more, about 2 us.
constexpr int kShortRow = 16384;
__global__ __launch_bounds__(kSampThreads) void short_row_stats_kernel(const float* __restrict__ logits, int V, float inv_temp,
                                                                       float* __restrict__ stats, const int* __restrict__ t_dev) {
  __shared__ float s_red[2][kSampWaves];
  if ((int)blockIdx.x >= dyn_tokens(t_dev, (int)gridDim.x)) return;  // (rows past the call's actual token count)
  const float* row = logits + (size_t)blockIdx.x * V;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  float m = -INFINITY;
  for (int i = tid; i < V; i += kSampThreads) m = fmaxf(m, row[i]);
  m = wave_max(m);
  if (lane == 0) s_red[0][w] = m;
  __syncthreads();
  m = s_red[0][0];
  for (int i = 1; i < kSampWaves; ++i) m = fmaxf(m, s_red[0][i]);
  float z = 0.0f;
  for (int i = tid; i < V; i += kSampThreads) z += __expf((row[i] - m) * inv_temp);
  z = wave_sum(z);
  if (lane == 0) s_red[1][w] = z;
  __syncthreads();
  if (tid == 0) {
    float t = 0.0f;
    for (int i = 0; i < kSampWaves; ++i) t += s_red[1][i];
    stats[(size_t)blockIdx.x * kSampStats] = m;
    stats[(size_t)blockIdx.x * kSampStats + 1] = t;
  }
}

__device__ __forceinline__ float wave_incl_scan_f32(float v, int lane) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const float t = __shfl_up(v, o);
    if (lane >= o) v += t;
  }
  return v;
}

// The walk of Eq. 3 over one tree by the whole workgroup. All threads: the target probability of every node's token under its
// parent's distribution. Then one wavefront, on values in LDS: child c of the surviving node is accepted when
// u_node[c] < p(c) / (1 - mass rejected so far at this node), which is what the repeated renormalisation amounts to; a token
// already rejected at this node has no mass left. The children of a node are found 64 nodes at a time by a ballot.
// Leaves the last node in *s_cur and the tokens rejected there, its children's, in s_rej[0 .. *s_nrej). `writer`: this
// workgroup writes the path (several may walk the same tree). Ends behind a barrier.
struct SampTree {
  int par[kMaxSel], tok[kMaxSel];
  float p[kMaxSel], u[kMaxSel];
};

template <bool SHORT>
__device__ __forceinline__ void sampled_walk(
    SampTree& s, int* s_rej, int* s_cur, int* s_nrej, bool writer, int lo, int n, const int32_t* __restrict__ parent,
    const int32_t* __restrict__ tok, const float* __restrict__ logits, int V, float inv_temp, const float* __restrict__ stats,
    const float* __restrict__ u_node, int32_t* __restrict__ my, int path_stride, int32_t* __restrict__ my_len,
    int32_t* __restrict__ status) {
  const int tid = threadIdx.x, lane = tid & 63, nthreads = blockDim.x;
  bool bad = false;
  for (int i = tid; i < n; i += nthreads) {
    int pa = parent[lo + i];
    int tk = tok[lo + i];
    if (i > 0 && (pa < 0 || pa >= i)) { bad = true; pa = 0; }
    float pr = 0.0f;
    if (i > 0) {
      if (tk < 0 || tk >= V) { bad = true; tk = -1; }  // an invalid token id is never accepted and removes no mass
      else {
        const size_t prow = (size_t)(lo + pa);
        const float* st = stats + prow * kSampStats;
        const float logit = logits[prow * V + tk];
        const float m = SHORT ? st[0] : stats_max(st);
        pr = __expf((logit - m) * inv_temp) / (SHORT ? st[1] : stats_sum(st, m, inv_temp));
      }
    }
    s.par[i] = i == 0 ? -1 : pa;
    s.tok[i] = tk;
    s.p[i] = pr;
    s.u[i] = u_node[lo + i];
  }
  if (bad && writer && status) atomicOr(status, ST_BAD_PARENT);
  if (writer)
    for (int i = tid; i < path_stride; i += nthreads) my[i] = i == 0 ? 0 : -1;
  __syncthreads();
  if (tid < 64) {
    int cur = 0, len = 1, nrej = 0;
    while (true) {
      float removed = 0.0f;
      nrej = 0;
      int nxt = -1;
      for (int base = cur + 1; base < n && nxt < 0; base += 64) {
        const int c0 = base + lane;
        unsigned long long kids = __ballot(c0 < n && s.par[c0] == cur);
        while (kids) {  // children in ascending order
          const int c = base + __ffsll((long long)kids) - 1;
          kids &= kids - 1;
          const int tk = s.tok[c];
          float pc = s.p[c];
          for (int r = 0; r < nrej; ++r)
            if (s_rej[r] == tk) pc = 0.0f;
          if (s.u[c] < pc / (1.0f - removed)) { nxt = c; break; }
          removed += pc;
          if (lane == 0) s_rej[nrej] = tk;
          wave_lds_fence();
          ++nrej;
        }
      }
      if (nxt < 0) break;
      cur = nxt;  // strictly increasing: the walk ends
      if (writer && lane == 0 && len < path_stride) my[len] = cur;
      ++len;
    }
    if (lane == 0) {
      if (writer) *my_len = len;
      *s_cur = cur;
      *s_nrej = nrej;
    }
  }
  __syncthreads();
}

// First node and size of tree b. An empty tree is taken for the one node at its offset; either way the nodes lie within the T of
// the call.
struct TreeSpan { int lo, n; };
__device__ __forceinline__ TreeSpan tree_span(const int32_t* __restrict__ tree_off, int b, int T) {
  int lo = tree_off[b], n = tree_off[b + 1] - lo;
  lo = lo < 0 ? 0 : (lo < T ? lo : T - 1);
  n = n < T - lo ? n : T - lo;
  return {lo, n < 1 ? 1 : (n > kMaxSel ? kMaxSel : n)};
}

// The final draw from the distribution at the last node with the rejected tokens removed, by inverting the cumulative sum at
// u_bonus: kSampWaves contiguous vocabulary segments are summed, the segment holding the target mass is cut into 64 contiguous
// pieces, the piece is walked. Lane l of a segment adds up elements 64j + l in ascending j, lane p of the pieces its own
// elements in ascending order: the order of every addition is fixed by the vocabulary size alone.

// segments start at multiples of 64
__device__ __forceinline__ int samp_segment(int V) { return (((V + kSampWaves - 1) / kSampWaves) + 63) & ~63; }

// which segment holds the target mass, and what of the target is left in it
__device__ __forceinline__ void pick_segment(const float* segsum, float u, int* segment, float* rem) {
  float total = 0.0f;
#pragma unroll
  for (int i = 0; i < kSampWaves; ++i) total += segsum[i];
  const float target = u * total;
  float before = 0.0f, last = 0.0f;
  int pick = -1;
  bool inside = false;
#pragma unroll
  for (int i = 0; i < kSampWaves; ++i) {
    if (!inside && segsum[i] > 0.0f) {
      pick = i;
      last = segsum[i];
      inside = target < before + last;
      if (!inside) before += last;
    }
  }
  // (rounding may leave the target past the last sum: the last non-empty segment takes it)
  if (pick >= 0 && !inside) before -= last;
  *segment = pick < 0 ? 0 : pick;
  *rem = target - before;
}

// Pieces of the segment at `base`, cl elements each, by a workgroup of 1024 threads: their exponentials go through LDS,
// LEN elements of every piece at a time, the first wavefront adds up one piece per lane and walks the one that holds
// `rem`. Returns the drawn token, in the first wavefront.
// A vocabulary of 151936 has pieces of 149: one round. Past 153600 logits there is a second one, and the drawn piece is evaluated again (all
// launches, four trees of 32 nodes, us, one workgroup per tree -> spread: 128256 logits 51.5 -> 38.6, 153600 60.6 -> 44.4, 153601 65.4 -> 56.0,
// 200064 76.9 -> 64.9, 262144 94.6 -> 81.1).
constexpr int kPieceLong = 150;
constexpr int piece_row(int len) { return len | 1; }                // odd: 64 lanes read 64 pieces without bank conflicts
template <int LEN>
__device__ __forceinline__ int draw_from_segment(float* s_piece, const int* s_rej, int nrej, const float* __restrict__ row, int V,
                                                 float m, float inv_temp, int base, int cl, float rem) {
  const int tid = threadIdx.x, lane = tid & 63;
  constexpr int ROW = piece_row(LEN);
  // running sums of every piece behind each kMark elements, so that the walk of the drawn piece need not start at its front
  constexpr int kMark = 16, kMarks = (LEN + kMark - 1) / kMark;
  static_assert(kMarks <= 64, "one mark per lane");
  __shared__ float s_mark[kMarks][64];
  constexpr int kLoads = (64 * LEN + kSampThreads - 1) / kSampThreads;
  float psum = 0.0f;
  for (int c0 = 0; c0 < cl; c0 += LEN) {
    const int cn = cl - c0 < LEN ? cl - c0 : LEN;
    const float per = 1.0f / (float)cn;
    float v[kLoads];
    int slot[kLoads];  // place in s_piece, -1: none
#pragma unroll
    for (int q = 0; q < kLoads; ++q) {
      const int f = tid + q * kSampThreads;  // (consecutive threads, consecutive elements where one round takes whole pieces)
      int piece = (int)((float)f * per);     // f / cn: below 2^14, so off by one at most
      if (piece * cn > f) --piece;
      if ((piece + 1) * cn <= f) ++piece;
      const int j = f - piece * cn, i = base + piece * cl + c0 + j;
      const bool in = f < 64 * cn;
      slot[q] = in ? (piece * ROW + j) | (i < V ? 0 : 1 << 30) : -1;
      v[q] = in && i < V ? row[i] : 0.0f;
    }
#pragma unroll
    for (int q = 0; q < kLoads; ++q)
      if (slot[q] >= 0) s_piece[slot[q] & ~(1 << 30)] = slot[q] >> 30 ? 0.0f : __expf((v[q] - m) * inv_temp);
    __syncthreads();
    for (int r = tid; r < nrej; r += kSampThreads) {
      const int at = s_rej[r] - base;
      if (at >= 0 && at < 64 * cl) {
        const int piece = at / cl, j = at - piece * cl - c0;
        if (j >= 0 && j < cn) s_piece[piece * ROW + j] = 0.0f;
      }
    }
    __syncthreads();
    if (tid < 64) {
      const float* mine = s_piece + lane * ROW;
      for (int j0 = 0, q = 0; j0 < cn; j0 += kMark, ++q) {
        float e[kMark];
#pragma unroll
        for (int u = 0; u < kMark; ++u) e[u] = j0 + u < cn ? mine[j0 + u] : 0.0f;
#pragma unroll
        for (int u = 0; u < kMark; ++u) psum += e[u];  // (trailing zeros leave a sum of non-negative terms as it is)
        if (cl <= LEN) s_mark[q][lane] = psum;
      }
    }
    if (cl > LEN) __syncthreads();
  }
  if (tid >= 64) return 0;
  const float incl = wave_incl_scan_f32(psum, lane);
  const unsigned long long hit = __ballot(psum > 0.0f && rem < incl);
  const unsigned long long any = __ballot(psum > 0.0f);
  int owner = -1;
  if (hit) owner = __ffsll((long long)hit) - 1;
  else if (any) owner = 63 - __clzll((long long)any);  // rounding: the last piece with mass takes it
  if (owner < 0) return 0;
  const float r2 = __shfl(rem - (incl - psum), owner);
  const int pb = base + owner * cl;
  int pick = -1;
  float run = 0.0f;
  bool inside = false;
  int first = 0;  // element the walk starts at, behind the last mark that the target lies past
  if (cl <= LEN) {
    wave_lds_fence();
    const int marks = (cl + kMark - 1) / kMark;
    const float mk = lane < marks ? s_mark[lane][owner] : 0.0f;
    const unsigned long long past = __ballot(lane < marks && mk > 0.0f && r2 < mk);
    if (past) {
      const int q = __ffsll((long long)past) - 1;
      first = q * kMark;
      if (q > 0) run = __shfl(mk, q - 1);
    }
  }
  for (int c0 = 0; c0 < cl && !inside; c0 += LEN) {
    const int cn = cl - c0 < LEN ? cl - c0 : LEN;
    const float* src = s_piece + owner * ROW;
    if (cl > LEN) {  // (LDS holds the last round: the owner's elements of this one again, by this wavefront)
      for (int j = lane; j < cn; j += 64) {
        const int i = pb + c0 + j;
        float e = i < V ? __expf((row[i] - m) * inv_temp) : 0.0f;
        for (int r = 0; r < nrej; ++r)
          if (s_rej[r] == i) e = 0.0f;
        s_piece[j] = e;
      }
      wave_lds_fence();
      src = s_piece;
    }
    for (int j0 = first; j0 < cn && !inside; j0 += 8) {
      float e[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) e[u] = j0 + u < cn ? src[j0 + u] : 0.0f;
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const bool take = !inside && e[u] > 0.0f;
        pick = take ? pb + c0 + j0 + u : pick;
        run = take ? run + e[u] : run;
        inside = take ? r2 < run : inside;
      }
    }
    if (cl > LEN) wave_lds_fence();
  }
  return pick < 0 ? 0 : pick;
}

// Rows of up to kOneDrawRow logits: one workgroup per tree walks, sums the segments, one per wavefront, and draws. PIECE: elements
// of a piece that one round takes, for rows of up to 1024 * PIECE logits.
// SHORT: statistics of short_row_stats_kernel; a segment is at most 16 loads per lane, and the code walked through counts.
// (One tree of 2 nodes, one of 32, four of 32, eight of 64, all launches, us, one workgroup -> spread as below: 50272 logits 20.4 -> 22.0,
// 22.1 -> 22.6, 26.1 -> 26.5, 46.8 -> 47.2; 65536 logits 21.0 -> 21.9, 22.9 -> 23.4, 29.0 -> 29.1, 55.5 -> 55.0; past that a lane takes a
// third batch of loads: 65537 logits 26.1 -> 23.7, 28.0 -> 25.8, 34.8 -> 31.3, 62.2 -> 59.6. Shorter pieces make shorter code: 32000
// logits, a tree of 32 nodes, 16.6 with pieces of 48, 17.0 with 64.)
constexpr int kOneDrawRow = 65536, kMidRow = 49152;
template <int PIECE>
__global__ __launch_bounds__(kSampThreads) void accept_sampled_kernel(
    const int32_t* __restrict__ tree_off, const int32_t* __restrict__ parent, const int32_t* __restrict__ tok,
    const float* __restrict__ logits, int V, float inv_temp, const float* __restrict__ stats,
    const float* __restrict__ u_node, const float* __restrict__ u_bonus, int T, int32_t* __restrict__ path, int path_stride,
    int32_t* __restrict__ path_len, int32_t* __restrict__ bonus, int32_t* __restrict__ status) {
  constexpr bool SHORT = PIECE * kSampWaves * 64 <= kShortRow;
  constexpr int kBatch = SHORT ? 4 : kStatsBatch;
  __shared__ SampTree s_tree;
  __shared__ int s_rej[kMaxSel];
  __shared__ float s_piece[64 * piece_row(PIECE)];
  __shared__ int s_cur, s_nrej;
  __shared__ float s_segsum[kSampWaves];
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const TreeSpan span = tree_span(tree_off, b, T);
  const int lo = span.lo, n = span.n;
  sampled_walk<SHORT>(s_tree, s_rej, &s_cur, &s_nrej, true, lo, n, parent, tok, logits, V, inv_temp, stats, u_node,
                     path + (size_t)b * path_stride, path_stride, path_len + b, status);
  const int cur = __builtin_amdgcn_readfirstlane(s_cur), nrej = __builtin_amdgcn_readfirstlane(s_nrej);
  const float* row = logits + (size_t)(lo + cur) * V;
  const float* st_cur = stats + (size_t)(lo + cur) * kSampStats;
  const float m = SHORT ? st_cur[0] : stats_max(st_cur);
  const int seg = samp_segment(V);
  const int sb = w * seg, se = sb + seg < V ? sb + seg : V;
  float acc = 0.0f;
  for (int i0 = sb; i0 < se; i0 += 64 * kBatch) {
    float e[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int i = i0 + u * 64 + lane;
      e[u] = i < se ? row[i] : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int i = i0 + u * 64 + lane;
      e[u] = i < se ? __expf((e[u] - m) * inv_temp) : 0.0f;
    }
    for (int r = 0; r < nrej; ++r) {  // (the same for the whole wavefront, and rarely inside this batch)
      const int at = __builtin_amdgcn_readfirstlane(s_rej[r]) - i0;
      if (at >= 0 && at < 64 * kBatch) {
#pragma unroll
        for (int u = 0; u < kBatch; ++u)
          if (u * 64 + lane == at) e[u] = 0.0f;
      }
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u) acc += e[u];  // (adding a zero leaves a sum of non-negative terms as it is)
  }
  acc = wave_sum(acc);
  if (lane == 0) s_segsum[w] = acc;
  __syncthreads();
  int segment;
  float rem;
  pick_segment(s_segsum, u_bonus[b], &segment, &rem);
  segment = __builtin_amdgcn_readfirstlane(segment);
  const int pick = draw_from_segment<PIECE>(s_piece, s_rej, nrej, row, V, m, inv_temp, segment * seg, seg >> 6, rem);
  if (tid == 0) bonus[b] = pick;
}

// Longer rows, in two launches. First one workgroup per (tree, segment): what bounds the sums is instruction issue, 149
// exponentials per lane and segment at a vocabulary of 151936, so they are spread over 16 CUs per tree instead of one, and
// over the four wavefronts of a workgroup, each a quarter of the 64-element blocks; the first wavefront then adds them up
// from LDS in order. Every workgroup walks the tree for itself, which costs no hand-off; the first one of a tree writes the
// path. A segment is summed relative to its own maximum, as nobody knows the row's where the walk ends in a leaf. What the draw
// needs goes behind the statistics of node b (kSampSeg, kSampSegMax, kSampCur).
constexpr int kSegThreads = 256;
constexpr int kSegBlocks = 152;  // blocks of 64 elements per round: one round up to a vocabulary of 155648
__global__ __launch_bounds__(kSegThreads) void accept_sampled_walk_kernel(
    const int32_t* __restrict__ tree_off, const int32_t* __restrict__ parent, const int32_t* __restrict__ tok,
    const float* __restrict__ logits, int V, float inv_temp, float* stats, const float* __restrict__ u_node,
    int T, int32_t* __restrict__ path, int path_stride, int32_t* __restrict__ path_len, int32_t* __restrict__ status) {
  constexpr int kWaves = kSegThreads / 64, kPer = kSegBlocks / kWaves;
  static_assert(kSegBlocks % kWaves == 0, "whole blocks per wavefront");
  __shared__ SampTree s_tree;
  __shared__ int s_rej[kMaxSel];
  __shared__ float s_e[kSegBlocks * 64], s_top[kWaves];
  __shared__ int s_cur, s_nrej;
  const int b = (int)blockIdx.x / kSampWaves, part = (int)blockIdx.x % kSampWaves;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const TreeSpan span = tree_span(tree_off, b, T);
  const int lo = span.lo, n = span.n;
  sampled_walk<false>(s_tree, s_rej, &s_cur, &s_nrej, part == 0, lo, n, parent, tok, logits, V, inv_temp, stats, u_node,
                      path + (size_t)b * path_stride, path_stride, path_len + b, status);
  const int cur = __builtin_amdgcn_readfirstlane(s_cur), nrej = __builtin_amdgcn_readfirstlane(s_nrej);
  const float* row = logits + (size_t)(lo + cur) * V;
  const int seg = samp_segment(V);
  const int sb = part * seg, se = sb + seg < V ? sb + seg : V;
  float m = -INFINITY, acc = 0.0f;  // of this segment: its own maximum, and the sum relative to it
  for (int c0 = sb; c0 < se; c0 += kSegBlocks * 64) {
    const int cn = se - c0 < kSegBlocks * 64 ? se - c0 : kSegBlocks * 64;
    float v[kPer];
    float top = m;
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int i = (u * kWaves + w) * 64 + lane;
      v[u] = i < cn ? row[c0 + i] : -INFINITY;
    }
#pragma unroll
    for (int u = 0; u < kPer; ++u) top = fmaxf(top, v[u]);
    top = wave_max(top);
    if (lane == 0) s_top[w] = top;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kWaves; ++u) top = fmaxf(top, s_top[u]);
    acc *= samp_exp(m, top, inv_temp);
    m = top;
#pragma unroll
    for (int u = 0; u < kPer; ++u) s_e[(u * kWaves + w) * 64 + lane] = samp_exp(v[u], m, inv_temp);
    __syncthreads();
    for (int r = tid; r < nrej; r += kSegThreads) {
      const int at = s_rej[r] - c0;
      if (at >= 0 && at < cn) s_e[at] = 0.0f;
    }
    __syncthreads();
    if (w == 0) {
      const int blocks = (cn + 63) >> 6;
#pragma unroll 8
      for (int q = 0; q < blocks; ++q) acc += s_e[q * 64 + lane];
    }
    __syncthreads();
  }
  if (w == 0) {
    acc = wave_sum(acc);
    float* out = stats + (size_t)b * kSampStats;
    if (lane == 0) {
      out[kSampSeg + part] = acc;
      out[kSampSegMax + part] = m;
      if (part == 0) out[kSampCur] = __int_as_float(cur);
    }
  }
}

// Second: one workgroup per tree draws from the segment that the sums pick. (Four trees of 32 nodes, vocabulary 151936: the
// walk and the draw 31 us in one workgroup per tree, 18 in these two launches; 8 and 10 us, of which 3 each are the launch.)
__global__ __launch_bounds__(kSampThreads) void accept_sampled_draw_kernel(
    const int32_t* __restrict__ tree_off, const int32_t* __restrict__ parent, const int32_t* __restrict__ tok,
    const float* __restrict__ logits, int V, float inv_temp, const float* __restrict__ stats, const float* __restrict__ u_bonus,
    int T, int32_t* __restrict__ bonus) {
  __shared__ int s_rej[kMaxSel];
  __shared__ float s_piece[64 * piece_row(kPieceLong)];
  __shared__ int s_nrej;
  const int b = blockIdx.x, tid = threadIdx.x;
  const TreeSpan span = tree_span(tree_off, b, T);
  const int lo = span.lo, n = span.n;
  const float* walked = stats + (size_t)b * kSampStats;
  const int cur = __builtin_amdgcn_readfirstlane(__float_as_int(walked[kSampCur]));
  if (tid == 0) s_nrej = 0;
  __syncthreads();
  for (int i = tid; i < n; i += kSampThreads) {  // the tokens rejected at the last node are its children's
    int pa = i == 0 ? -1 : parent[lo + i];
    if (i > 0 && (pa < 0 || pa >= i)) pa = 0;
    const int tk = tok[lo + i];
    if (pa == cur) s_rej[atomicAdd(&s_nrej, 1)] = tk < 0 || tk >= V ? -1 : tk;
  }
  const float m = stats_max(walked + kSampSegMax);
  float segsum[kSampWaves];
#pragma unroll
  for (int i = 0; i < kSampWaves; ++i) segsum[i] = walked[kSampSeg + i] * samp_exp(walked[kSampSegMax + i], m, inv_temp);
  int segment;
  float rem;
  pick_segment(segsum, u_bonus[b], &segment, &rem);
  segment = __builtin_amdgcn_readfirstlane(segment);
  __syncthreads();
  const int nrej = __builtin_amdgcn_readfirstlane(s_nrej);
  const int seg = samp_segment(V);
  const int pick = draw_from_segment<kPieceLong>(s_piece, s_rej, nrej, logits + (size_t)(lo + cur) * V, V, m, inv_temp,
                                                 segment * seg, seg >> 6, rem);
  if (tid == 0) bonus[b] = pick;
}

// the launches of acceptance under sampling on `stats`, [T][kSampStats] floats of scratch
int launch_accept_sampled(const int32_t* tree_off, const int32_t* parent, const int32_t* tok, const float* logits, int V,
                          float inv_temp, float* stats, const float* u_node, const float* u_bonus, int B, int T, int32_t* path,
                          int path_stride, int32_t* path_len, int32_t* bonus, int32_t* status, const int32_t* t_dev, hipStream_t s) {
  // An infinite temperature: the smallest factor instead of 0, whose product with the -inf of masked logits, and of what the kernels take for
  // places past a row's end, is no number. Any two logits less than 1e37 apart still weigh the same. (A test for -inf at every exponential
  // takes 2 us of 33 at four trees of 32 nodes, vocabulary 151936.)
  if (inv_temp == 0.0f) inv_temp = 1.40129846e-45f;
  const bool one_draw = V <= kOneDrawRow || B > T;  // (more trees than nodes, so some of them empty: no room to hand over)
  if (V <= kShortRow) {
    hipLaunchKernelGGL(short_row_stats_kernel, dim3(T), dim3(kSampThreads), 0, s, logits, V, inv_temp, stats, t_dev);
  } else {
    hipLaunchKernelGGL(row_stats_kernel, dim3(T * kStatsWgs), dim3(kStatsThreads), 0, s, logits, V, inv_temp, stats, T, t_dev, tree_off,
                       parent, B, one_draw ? 0 : 1);
  }
  int rc = launch_status("softmax statistics kernels");
  if (rc) return rc;
#define EVICT_ONE_DRAW(ROW_)                                                                                                       \
  hipLaunchKernelGGL(accept_sampled_kernel<(ROW_) / (kSampWaves * 64)>, dim3(B), dim3(kSampThreads), 0, s, tree_off, parent, tok,   \
                     logits, V, inv_temp, stats, u_node, u_bonus, T, path, path_stride, path_len, bonus, status)
  if (one_draw) {
    if (V <= kShortRow) EVICT_ONE_DRAW(kShortRow);
    else if (V <= kMidRow) EVICT_ONE_DRAW(kMidRow);
    else EVICT_ONE_DRAW(kOneDrawRow);
    return launch_status("accept_sampled_kernel");
  }
#undef EVICT_ONE_DRAW
  hipLaunchKernelGGL(accept_sampled_walk_kernel, dim3(B * kSampWaves), dim3(kSegThreads), 0, s, tree_off, parent, tok, logits, V, inv_temp,
                     stats, u_node, T, path, path_stride, path_len, status);
  hipLaunchKernelGGL(accept_sampled_draw_kernel, dim3(B), dim3(kSampThreads), 0, s, tree_off, parent, tok, logits, V, inv_temp, stats,
                     u_bonus, T, bonus);
  return launch_status("accept_sampled_draw_kernel");
}

constexpr int kUnionThreads = 1024;  // >= the largest supported E: one expert per thread in the scan

__global__ __launch_bounds__(kUnionThreads) void expert_union_kernel(
    const int32_t* __restrict__ topk_idx, int T, int k, int E, int use_masks, int32_t* __restrict__ union_ids,
    int32_t* __restrict__ union_count, int32_t* __restrict__ hist, int32_t* __restrict__ offsets,
    int32_t* __restrict__ perm, int32_t* __restrict__ inv, int32_t* __restrict__ status) {
  extern __shared__ __attribute__((aligned(8))) int s_mem[];
  expert_union_body(s_mem, topk_idx, T, k, E, use_masks, union_ids, union_count, hist, offsets, perm, inv, status, nullptr,
                    nullptr);
}

typedef __attribute__((ext_vector_type(4))) unsigned int probe_u32x4;

// Streaming read: 512 workgroups x 256 threads, each thread keeps 8 independent 16-byte loads in flight.
__global__ __launch_bounds__(256) void probe_read_kernel(const probe_u32x4* __restrict__ src, size_t n16, unsigned* __restrict__ sink) {
  const size_t per_wg = (n16 + gridDim.x - 1) / gridDim.x;
  const size_t lo = per_wg * blockIdx.x;
  size_t hi = lo + per_wg;
  hi = hi > n16 ? n16 : hi;
  probe_u32x4 acc = {0, 0, 0, 0};
  for (size_t i = lo + threadIdx.x; i < hi; i += 256 * 8) {
    probe_u32x4 v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const size_t idx = i + (size_t)j * 256;
      v[j] = idx < hi ? __builtin_nontemporal_load(src + idx) : probe_u32x4{0, 0, 0, 0};
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) acc ^= v[j];
  }
  if ((acc[0] ^ acc[1] ^ acc[2] ^ acc[3]) == 0x9E3779B9u) sink[threadIdx.x & 3] = acc[0];  // keeps the loads alive
}

__global__ __launch_bounds__(256) void probe_copy_kernel(const probe_u32x4* __restrict__ src, probe_u32x4* __restrict__ dst, size_t n16) {
  const size_t per_wg = (n16 + gridDim.x - 1) / gridDim.x;
  const size_t lo = per_wg * blockIdx.x;
  size_t hi = lo + per_wg;
  hi = hi > n16 ? n16 : hi;
  for (size_t i = lo + threadIdx.x; i < hi; i += 256 * 4) {
    probe_u32x4 v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const size_t idx = i + (size_t)j * 256;
      if (idx < hi) v[j] = src[idx];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const size_t idx = i + (size_t)j * 256;
      if (idx < hi) dst[idx] = v[j];
    }
  }
}

// One workgroup per destination row. The row's tree is found by counting, a wavefront at a time, the trees that end at or
// before it; rows that are whole 16-byte pieces on both sides move as such (W = uint4), the rest as 4-byte words.
template <typename W>
__global__ __launch_bounds__(128) void gather_rows_kernel(const W* __restrict__ src, W* __restrict__ dst, int row_words,
                                   const int32_t* __restrict__ tree_off, const int32_t* __restrict__ new_tree_off,
                                   const int32_t* __restrict__ keep, int B) {
  const int r = blockIdx.x;  // destination row
  if (r >= new_tree_off[B]) return;
  const int node = keep[r];
  int b = 0;
  for (int b0 = 0; b0 + 1 < B; b0 += 64) {
    const int t = b0 + lane_id();
    const unsigned long long m = __ballot(t + 1 < B && new_tree_off[t + 1] <= r);
    b += __popcll(m);
    if (m != ~0ull) break;  // the offsets ascend
  }
  const int s = tree_off[b] + node;
  for (int i = threadIdx.x; i < row_words; i += 128) dst[(size_t)r * row_words + i] = src[(size_t)s * row_words + i];
}

// Commit of the accepted path to the KV cache: the j-th accepted node of sequence b (depth j, so
// its key was rotated at position ctx_len[b] + j) becomes cache row ctx_len[b] + j of every KV
// head. Grid (path position, sequence); rows are copied as 4-byte words. Rows that would fall
// past the cache capacity are dropped and the new length is clamped.
constexpr int kCommitLayers = 64;  // layers per launch (their pointers travel as a kernel argument)
struct KvLayerPtrs {
  const uint32_t* k_new[kCommitLayers];
  const uint32_t* v_new[kCommitLayers];
  uint32_t* k_cache[kCommitLayers];
  uint32_t* v_cache[kCommitLayers];
};

__global__ __launch_bounds__(256) void kv_commit_kernel(
    const KvLayerPtrs lp, int Hkv, int head_words,
    const int32_t* __restrict__ tree_off, const int32_t* __restrict__ path, int path_stride,
    const int32_t* __restrict__ path_len, long long seq_words, long long head_stride_words,
    const int32_t* __restrict__ ctx_len, int capacity, int32_t* __restrict__ ctx_len_out, int32_t* __restrict__ status,
    const KvPaging pg) {
  const int j = blockIdx.x, b = blockIdx.y, layer = blockIdx.z;
  const uint32_t* __restrict__ k_new = lp.k_new[layer];
  const uint32_t* __restrict__ v_new = lp.v_new[layer];
  uint32_t* __restrict__ k_cache = lp.k_cache[layer];
  uint32_t* __restrict__ v_cache = lp.v_cache[layer];
  int len = path_len[b];
  // an accepted path longer than the rows `path` holds (evict_accept_path truncates it) cannot be committed in
  // full: the rows that are there are committed, the length advances by that many, and the call is flagged
  const bool trunc = len > path_stride;
  len = len < 0 ? 0 : (trunc ? path_stride : len);
  int L = ctx_len[b];
  const bool badL = L < 0 || L > capacity;
  L = L < 0 ? 0 : (L > capacity ? capacity : L);
  const int room = capacity - L;
  if (j == 0 && layer == 0 && threadIdx.x == 0) {
    ctx_len_out[b] = L + (len < room ? len : room);
    if (status && (badL || len > room)) atomicOr(status, ST_BAD_CTXLEN);
    if (status && trunc) atomicOr(status, ST_PATH_TRUNCATED);
  }
  if (j >= len || j >= room) return;
  const int n = tree_off[b + 1] - tree_off[b];
  const int node = path[(size_t)b * path_stride + j];
  if (node < 0 || node >= n) {
    if (status && threadIdx.x == 0) atomicOr(status, ST_BAD_PARENT);
    return;
  }
  const size_t src = (size_t)(tree_off[b] + node) * Hkv * head_words;
  const int row_words = Hkv * head_words;
  // start of the destination row of head 0: contiguous cache, or (paged: seq_words is the distance
  // between pages) the page the table names for position L + j
  size_t row0 = (size_t)b * seq_words + (size_t)(L + j) * head_words;
  if (pg.table) {
    const int pos = L + j;
    const int pid = pg.table[(size_t)b * pg.table_stride + (pos >> pg.page_shift)];
    if ((unsigned)pid >= (unsigned)pg.n_pages) {  // never write through a bad page id
      if (status && threadIdx.x == 0) atomicOr(status, ST_BAD_PAGE);
      return;
    }
    row0 = (size_t)pid * seq_words + (size_t)(pos & ((1 << pg.page_shift) - 1)) * head_words;
  }
  for (int i = threadIdx.x; i < row_words; i += 256) {
    const int h = i / head_words, c = i - h * head_words;
    const size_t dst = row0 + (size_t)h * head_stride_words + c;
    k_cache[dst] = k_new[src + i];
    v_cache[dst] = v_new[src + i];
  }
}

}  // namespace

int union_mask_plan(int T, int k, int E, size_t* lds_bytes) {
  const int P = T * k;
  const size_t words = (size_t)(T + 63) / 64;
  size_t lds = sizeof(int) * union_lds_ints(P, E);
  const size_t mask_bytes = union_mask_bytes(E, (int)words), before_bytes = union_before_bytes(E, (int)words);
  const int use_masks = lds + mask_bytes + before_bytes <= 60 * 1024 ? 2 : (lds + mask_bytes <= 60 * 1024 ? 1 : 0);
  if (use_masks) lds += mask_bytes;
  if (use_masks == 2) lds += before_bytes;
  *lds_bytes = lds;
  return use_masks;
}

}  // namespace evict

using namespace evict;

// ---- scratch of the allocation-free entry point (evict_accept_path_sampled_noalloc) ----
// Per-node softmax statistics [EVICT_NOALLOC_MAX_NODES][EVICT_SAMP_STATS] floats. Every GPU the library runs on holds its
// own copy of this array until the process ends. In host code the array's name is only a stand-in: the
// device address is looked up once per device and kept; kernels and copies use that pointer.
static __device__ __align__(256) float scratch[EVICT_NOALLOC_MAX_NODES * EVICT_SAMP_STATS];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
float* g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device (looked up on the first call on that device).
int scratch_address(float** out) {
  int dev = -1;
  EVICT_HIP_CHECK(hipGetDevice(&dev));
  EVICT_REQUIRE(dev >= 0 && dev < kMaxDevices, EVICT_E_UNSUPPORTED, "device ordinal %d outside [0, %d)", dev, kMaxDevices);
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    EVICT_HIP_CHECK(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    EVICT_REQUIRE(p != nullptr, EVICT_E_HIP, "hipGetSymbolAddress returned a null address for the static scratch");
    g_scratch_ptr[dev] = static_cast<float*>(p);
  }
  *out = g_scratch_ptr[dev];
  return EVICT_OK;
}
}  // namespace

extern "C" {

int evict_version(void) { return 1; }

const char* evict_last_error(void) { return g_err; }

int evict_validate_trees_host(const int32_t* tree_off, const int32_t* parent, int B, int max_nodes) {
  EVICT_REQUIRE(tree_off && parent, EVICT_E_INVALID, "null tree arrays");
  EVICT_REQUIRE(B >= 1, EVICT_E_INVALID, "B must be >= 1 (got %d)", B);
  EVICT_REQUIRE(tree_off[0] == 0, EVICT_E_INVALID, "tree_off[0] must be 0");
  for (int b = 0; b < B; ++b) {
    const int lo = tree_off[b], n = tree_off[b + 1] - lo;
    EVICT_REQUIRE(n >= 1, EVICT_E_INVALID, "tree %d has %d nodes", b, n);
    EVICT_REQUIRE(n <= max_nodes, EVICT_E_INVALID, "tree %d has %d nodes, limit %d", b, n, max_nodes);
    EVICT_REQUIRE(parent[lo] == -1, EVICT_E_INVALID, "tree %d: root parent must be -1", b);
    for (int i = 1; i < n; ++i)
      EVICT_REQUIRE(parent[lo + i] >= 0 && parent[lo + i] < i, EVICT_E_INVALID,
                    "tree %d: parent[%d]=%d is not in [0,%d)", b, i, parent[lo + i], i);
  }
  return EVICT_OK;
}

static int select_prefix_impl(const char* who, evict_ctx* ctx, const int32_t* tree_off, const int32_t* parent, const float* node_prob, int B,
                              int T, const float* cost, float rho, int Kmax, int32_t* k_star, int32_t* keep,
                              int32_t* new_parent, int32_t* new_tree_off, float* est_len, int32_t* order,
                              float* prefix_sum, void* stream) {
  EVICT_REQUIRE(tree_off && parent && node_prob && k_star && keep && new_parent && new_tree_off && est_len,
                EVICT_E_INVALID, "%s: null pointer argument", who);
  EVICT_REQUIRE(B >= 1 && T >= B, EVICT_E_INVALID, "%s: need B >= 1 and T >= B (B=%d, T=%d)", who, B, T);
  EVICT_REQUIRE(Kmax >= 1, EVICT_E_INVALID, "%s: Kmax must be >= 1 (got %d)", who, Kmax);
  EVICT_REQUIRE(T <= B * (int64_t)EVICT_MAX_SELECT_NODES, EVICT_E_UNSUPPORTED, "%s: more than %d nodes per tree", who,
                EVICT_MAX_SELECT_NODES);
  hipStream_t s = (hipStream_t)stream;
  int32_t* status = ctx ? ctx->status : nullptr;
  const int single = B == 1;
  if (B == 1 && T <= 64) {  // one small tree: the single-wavefront register kernel
    hipLaunchKernelGGL(select_prefix_wave_kernel, dim3(1), dim3(64), 0, s, parent, node_prob, cost, Kmax, T, rho, k_star,
                       est_len, order, prefix_sum, keep, new_parent, new_tree_off, status);
    return launch_status("select_prefix_wave_kernel");
  }
  const int sel_threads = T > (int64_t)64 * B ? kSelThreads : kSelThreadsSmall;
  hipLaunchKernelGGL(select_prefix_kernel, dim3(B), dim3(sel_threads), 0, s, tree_off, parent, node_prob, cost, Kmax,
                     k_star, est_len, order, prefix_sum, new_parent /* rank workspace */, single, keep, new_parent,
                     new_tree_off, single ? T : 0, rho, status);
  int rc = launch_status("select_prefix_kernel");
  if (rc) return rc;
  if (!single) {
    hipLaunchKernelGGL(compact_batch_kernel, dim3(1), dim3(kCompactThreads), 0, s, tree_off, parent, k_star, B,
                       new_parent, keep, new_parent, new_tree_off);
    rc = launch_status("compact_batch_kernel");
  }
  return rc;
}

int evict_select_prefix(evict_ctx* ctx, const int32_t* tree_off, const int32_t* parent, const float* node_prob, int B,
                        int T, const float* cost, int Kmax, int32_t* k_star, int32_t* keep, int32_t* new_parent,
                        int32_t* new_tree_off, float* est_len, int32_t* order, float* prefix_sum, void* stream) {
  EVICT_REQUIRE(cost, EVICT_E_INVALID, "evict_select_prefix: null cost table");
  return select_prefix_impl("evict_select_prefix", ctx, tree_off, parent, node_prob, B, T, cost, -1.0f, Kmax, k_star, keep,
                            new_parent, new_tree_off, est_len, order, prefix_sum, stream);
}

int evict_select_prefix_coverage(evict_ctx* ctx, const int32_t* tree_off, const int32_t* parent, const float* node_prob, int B,
                                 int T, float rho, int Kmax, int32_t* k_star, int32_t* keep, int32_t* new_parent,
                                 int32_t* new_tree_off, float* est_len, int32_t* order, float* prefix_sum, void* stream) {
  EVICT_REQUIRE(rho >= 0.0f && rho <= 1.0f, EVICT_E_INVALID, "evict_select_prefix_coverage: rho=%g outside [0, 1]", (double)rho);
  return select_prefix_impl("evict_select_prefix_coverage", ctx, tree_off, parent, node_prob, B, T, nullptr, rho, Kmax, k_star,
                            keep, new_parent, new_tree_off, est_len, order, prefix_sum, stream);
}

int evict_accept_path(evict_ctx*, const int32_t* tree_off, const int32_t* parent, const int32_t* draft_tok,
                      const int32_t* target_next, int B, int32_t* path, int path_stride, int32_t* path_len,
                      int32_t* bonus_tok, void* stream) {
  EVICT_REQUIRE(tree_off && parent && draft_tok && target_next && path && path_len && bonus_tok, EVICT_E_INVALID,
                "evict_accept_path: null pointer argument");
  EVICT_REQUIRE(B >= 1, EVICT_E_INVALID, "evict_accept_path: B must be >= 1 (got %d)", B);
  EVICT_REQUIRE(path_stride >= 1, EVICT_E_INVALID, "evict_accept_path: path_stride must be >= 1");
  hipLaunchKernelGGL(accept_path_kernel, dim3(B), dim3(64), 0, (hipStream_t)stream, tree_off, parent, draft_tok,
                     target_next, path, path_stride, path_len, bonus_tok);
  return launch_status("accept_path_kernel");
}

int evict_expert_union(evict_ctx* ctx, const int32_t* topk_idx, int T, int k, int E, int32_t* union_ids,
                       int32_t* union_count, int32_t* hist, int32_t* offsets, int32_t* perm, int32_t* inv,
                       void* stream) {
  EVICT_REQUIRE(topk_idx && union_ids && union_count && hist && offsets && perm && inv, EVICT_E_INVALID,
                "evict_expert_union: null pointer argument");
  EVICT_REQUIRE(T >= 1 && k >= 1 && E >= 1, EVICT_E_INVALID, "evict_expert_union: T, k, E must be >= 1");
  EVICT_REQUIRE(k <= E, EVICT_E_INVALID, "evict_expert_union: k=%d exceeds E=%d", k, E);
  EVICT_REQUIRE((int64_t)T * k <= 8192 && E <= 1024, EVICT_E_UNSUPPORTED,
                "evict_expert_union: T*k=%lld (limit 8192), E=%d (limit 1024)", (long long)T * k, E);
  size_t lds;
  const int use_masks = union_mask_plan(T, k, E, &lds);
  hipLaunchKernelGGL(expert_union_kernel, dim3(1), dim3(kUnionThreads), lds, (hipStream_t)stream, topk_idx, T, k, E,
                     use_masks, union_ids, union_count, hist, offsets, perm, inv, ctx ? ctx->status : nullptr);
  return launch_status("expert_union_kernel");
}

int evict_probe_read(const void* src, size_t bytes, void* sink, void* stream) {
  EVICT_REQUIRE(src && sink && bytes > 0 && bytes % 16 == 0 && aligned16(src), EVICT_E_INVALID,
                "evict_probe_read: need non-null 16-byte aligned src, sink, and bytes a positive multiple of 16");
  hipLaunchKernelGGL(probe_read_kernel, dim3(2048), dim3(256), 0, (hipStream_t)stream, (const probe_u32x4*)src, bytes / 16,
                     (unsigned*)sink);
  return launch_status("probe_read_kernel");
}

int evict_probe_copy(const void* src, void* dst, size_t bytes, void* stream) {
  EVICT_REQUIRE(src && dst && bytes > 0 && bytes % 16 == 0 && aligned16(src) && aligned16(dst), EVICT_E_INVALID,
                "evict_probe_copy: need non-null 16-byte aligned pointers and bytes a positive multiple of 16");
  hipLaunchKernelGGL(probe_copy_kernel, dim3(2048), dim3(256), 0, (hipStream_t)stream, (const probe_u32x4*)src,
                     (probe_u32x4*)dst, bytes / 16);
  return launch_status("probe_copy_kernel");
}

int evict_gather_rows(const void* src, void* dst, int row_bytes, const int32_t* tree_off, const int32_t* new_tree_off,
                      const int32_t* keep, int B, int T, void* stream) {
  EVICT_REQUIRE(src && dst && tree_off && new_tree_off && keep, EVICT_E_INVALID, "evict_gather_rows: null pointer");
  EVICT_REQUIRE(row_bytes > 0 && row_bytes % 4 == 0, EVICT_E_INVALID, "evict_gather_rows: row_bytes must be a positive multiple of 4");
  EVICT_REQUIRE(B >= 1 && T >= 1, EVICT_E_INVALID, "evict_gather_rows: B, T must be >= 1");
  EVICT_REQUIRE(src != dst, EVICT_E_INVALID, "evict_gather_rows: in-place gather is not supported");
  if (row_bytes % 16 == 0 && aligned16(src) && aligned16(dst))
    hipLaunchKernelGGL(gather_rows_kernel<uint4>, dim3(T), dim3(128), 0, (hipStream_t)stream, (const uint4*)src, (uint4*)dst,
                       row_bytes / 16, tree_off, new_tree_off, keep, B);
  else
    hipLaunchKernelGGL(gather_rows_kernel<uint32_t>, dim3(T), dim3(128), 0, (hipStream_t)stream, (const uint32_t*)src,
                       (uint32_t*)dst, row_bytes / 4, tree_off, new_tree_off, keep, B);
  return launch_status("gather_rows_kernel");
}

int evict_accept_path_sampled(evict_ctx* ctx, const int32_t* tree_off, const int32_t* parent, const int32_t* draft_tok,
                              const float* logits, int vocab, float temperature, const float* u_node, const float* u_bonus,
                              int B, int T, int32_t* path, int path_stride, int32_t* path_len, int32_t* bonus_tok,
                              void* stream) {
  EVICT_REQUIRE(ctx && tree_off && parent && draft_tok && logits && u_node && u_bonus && path && path_len && bonus_tok,
                EVICT_E_INVALID, "evict_accept_path_sampled: null pointer argument");
  EVICT_REQUIRE(B >= 1 && B <= ctx->max_batch, EVICT_E_INVALID, "evict_accept_path_sampled: B=%d outside [1,%d]", B, ctx->max_batch);
  EVICT_REQUIRE(T >= 1 && T <= ctx->max_tokens, EVICT_E_INVALID, "evict_accept_path_sampled: T=%d outside [1,%d]", T, ctx->max_tokens);
  EVICT_REQUIRE(vocab >= 1, EVICT_E_INVALID, "evict_accept_path_sampled: vocab must be >= 1");
  EVICT_REQUIRE(temperature > 0.0f && temperature == temperature, EVICT_E_INVALID,
                "evict_accept_path_sampled: temperature must be > 0 (use evict_accept_path for the greedy rule)");
  EVICT_REQUIRE(path_stride >= 1, EVICT_E_INVALID, "evict_accept_path_sampled: path_stride must be >= 1");
  const float inv_temp = 1.0f / temperature;
  hipStream_t s = (hipStream_t)stream;
  return launch_accept_sampled(tree_off, parent, draft_tok, logits, vocab, inv_temp, ctx->samp_stats, u_node, u_bonus, B, T, path,
                               path_stride, path_len, bonus_tok, ctx->status, ctx->t_dev, s);
}

int evict_accept_path_sampled_noalloc(evict_ctx* ctx, const int32_t* tree_off, const int32_t* parent, const int32_t* draft_tok,
                                      const float* logits, int vocab, float temperature, const float* u_node,
                                      const float* u_bonus, int B, int T, int32_t* path, int path_stride, int32_t* path_len,
                                      int32_t* bonus_tok, void* stream) {
  EVICT_REQUIRE(tree_off && parent && draft_tok && logits && u_node && u_bonus && path && path_len && bonus_tok,
                EVICT_E_INVALID, "evict_accept_path_sampled_noalloc: null pointer argument");
  EVICT_REQUIRE(B >= 1 && B <= 65535, EVICT_E_INVALID, "evict_accept_path_sampled_noalloc: B=%d outside [1, 65535]", B);
  EVICT_REQUIRE(T >= B, EVICT_E_INVALID, "evict_accept_path_sampled_noalloc: T=%d is smaller than B=%d", T, B);
  EVICT_REQUIRE(T <= EVICT_NOALLOC_MAX_NODES, EVICT_E_UNSUPPORTED,
                "evict_accept_path_sampled_noalloc: T=%d exceeds the static scratch of %d nodes (use evict_accept_path_sampled)", T,
                EVICT_NOALLOC_MAX_NODES);
  EVICT_REQUIRE(vocab >= 1, EVICT_E_INVALID, "evict_accept_path_sampled_noalloc: vocab must be >= 1");
  EVICT_REQUIRE(temperature > 0.0f && temperature == temperature, EVICT_E_INVALID,
                "evict_accept_path_sampled_noalloc: temperature must be > 0 (use evict_accept_path for the greedy rule)");
  EVICT_REQUIRE(path_stride >= 1, EVICT_E_INVALID, "evict_accept_path_sampled_noalloc: path_stride must be >= 1");
  float* stats = nullptr;
  int rc = scratch_address(&stats);
  if (rc) return rc;
  const float inv_temp = 1.0f / temperature;
  hipStream_t s = (hipStream_t)stream;
  // (what a call reads of the statistics it has written before: nothing has to start at zero)
  return launch_accept_sampled(tree_off, parent, draft_tok, logits, vocab, inv_temp, stats, u_node, u_bonus, B, T, path, path_stride,
                               path_len, bonus_tok, ctx ? ctx->status : nullptr, ctx ? ctx->t_dev : nullptr, s);
}

static int kv_commit_impl(const char* who, evict_ctx* ctx, int dtype, int Hkv, int D, const void* const* k_new,
                          const void* const* v_new, int n_layers, const int32_t* tree_off, const int32_t* path, int path_stride,
                          const int32_t* path_len, void* const* k_caches, void* const* v_caches, int64_t kv_seq_stride,
                          int64_t kv_head_stride, const int32_t* ctx_len, int capacity, int32_t* ctx_len_out, int B,
                          void* stream, const KvPaging pg = KvPaging{nullptr, 0, 0, 0}) {
  EVICT_REQUIRE(k_new && v_new && tree_off && path && path_len && k_caches && v_caches && ctx_len && ctx_len_out,
                EVICT_E_INVALID, "%s: null pointer argument", who);
  EVICT_REQUIRE(dtype == EVICT_F32 || dtype == EVICT_BF16, EVICT_E_INVALID, "%s: unknown dtype %d", who, dtype);
  EVICT_REQUIRE(n_layers >= 1, EVICT_E_INVALID, "%s: n_layers=%d", who, n_layers);
  EVICT_REQUIRE(B >= 1 && B <= 65535 && Hkv >= 1 && D >= 1 && path_stride >= 1 && path_stride <= EVICT_MAX_SELECT_NODES,
                EVICT_E_INVALID, "%s: B, Hkv, D, path_stride out of range", who);
  const int eb = dtype == EVICT_BF16 ? 2 : 4;
  EVICT_REQUIRE((D * eb) % 4 == 0, EVICT_E_INVALID, "%s: a head row must be a multiple of 4 bytes", who);
  if (pg.table) {
    const int64_t page = (int64_t)1 << pg.page_shift;
    EVICT_REQUIRE(capacity >= 1 && (int64_t)pg.table_stride * page >= capacity, EVICT_E_INVALID,
                  "%s: a table row covers %lld positions, capacity is %d", who, (long long)pg.table_stride * page, capacity);
    EVICT_REQUIRE(kv_head_stride >= page * D && kv_seq_stride >= kv_head_stride * Hkv && (kv_head_stride * eb) % 4 == 0 &&
                      (kv_seq_stride * eb) % 4 == 0,
                  EVICT_E_INVALID, "%s: page strides do not hold page_size=%lld rows per head", who, (long long)page);
  } else {
    EVICT_REQUIRE(capacity >= 1 && kv_head_stride >= (int64_t)capacity * D && (kv_head_stride * eb) % 4 == 0 &&
                      (kv_seq_stride * eb) % 4 == 0 && (B == 1 || kv_seq_stride >= kv_head_stride * Hkv),
                  EVICT_E_INVALID, "%s: cache strides do not hold capacity=%d rows per head", who, capacity);
  }
  EVICT_REQUIRE(ctx_len_out != ctx_len, EVICT_E_INVALID, "%s: ctx_len_out must not alias ctx_len", who);
  for (int l = 0; l < n_layers; ++l)
    EVICT_REQUIRE(k_new[l] && v_new[l] && k_caches[l] && v_caches[l], EVICT_E_INVALID, "%s: null pointer for layer %d", who, l);
  const int head_words = D * eb / 4;
  for (int l0 = 0; l0 < n_layers; l0 += kCommitLayers) {
    const int nl = n_layers - l0 < kCommitLayers ? n_layers - l0 : kCommitLayers;
    KvLayerPtrs lp = {};
    for (int l = 0; l < nl; ++l) {
      lp.k_new[l] = (const uint32_t*)k_new[l0 + l];
      lp.v_new[l] = (const uint32_t*)v_new[l0 + l];
      lp.k_cache[l] = (uint32_t*)k_caches[l0 + l];
      lp.v_cache[l] = (uint32_t*)v_caches[l0 + l];
    }
    hipLaunchKernelGGL(kv_commit_kernel, dim3(path_stride, B, nl), dim3(256), 0, (hipStream_t)stream, lp, Hkv, head_words,
                       tree_off, path, path_stride, path_len, (long long)(kv_seq_stride * eb / 4),
                       (long long)(kv_head_stride * eb / 4), ctx_len, capacity, ctx_len_out, ctx ? ctx->status : nullptr, pg);
    int rc = launch_status("kv_commit_kernel");
    if (rc) return rc;
  }
  return EVICT_OK;
}

int evict_kv_commit(evict_ctx* ctx, int dtype, int Hkv, int D, const void* k_new, const void* v_new, const int32_t* tree_off,
                    const int32_t* path, int path_stride, const int32_t* path_len, void* k_cache, void* v_cache,
                    int64_t kv_seq_stride, int64_t kv_head_stride, const int32_t* ctx_len, int capacity, int32_t* ctx_len_out,
                    int B, void* stream) {
  return kv_commit_impl("evict_kv_commit", ctx, dtype, Hkv, D, &k_new, &v_new, 1, tree_off, path, path_stride, path_len,
                        &k_cache, &v_cache, kv_seq_stride, kv_head_stride, ctx_len, capacity, ctx_len_out, B, stream);
}

int evict_kv_commit_stack(evict_ctx* ctx, int dtype, int Hkv, int D, const void* const* k_new, const void* const* v_new,
                          int n_layers, const int32_t* tree_off, const int32_t* path, int path_stride, const int32_t* path_len,
                          void* const* k_caches, void* const* v_caches, int64_t kv_seq_stride, int64_t kv_head_stride,
                          const int32_t* ctx_len, int capacity, int32_t* ctx_len_out, int B, void* stream) {
  return kv_commit_impl("evict_kv_commit_stack", ctx, dtype, Hkv, D, k_new, v_new, n_layers, tree_off, path, path_stride,
                        path_len, k_caches, v_caches, kv_seq_stride, kv_head_stride, ctx_len, capacity, ctx_len_out, B, stream);
}

int evict_kv_commit_stack_paged(evict_ctx* ctx, int dtype, int Hkv, int D, const void* const* k_new, const void* const* v_new,
                                int n_layers, const int32_t* tree_off, const int32_t* path, int path_stride,
                                const int32_t* path_len, void* const* k_pools, void* const* v_pools, int64_t page_stride,
                                int64_t kv_head_stride, const int32_t* block_table, int table_stride, int page_size, int n_pages,
                                const int32_t* ctx_len, int capacity, int32_t* ctx_len_out, int B, void* stream) {
  EVICT_REQUIRE(block_table, EVICT_E_INVALID, "evict_kv_commit_stack_paged: null block table");
  EVICT_REQUIRE(page_size >= 1 && page_size <= 65536 && (page_size & (page_size - 1)) == 0, EVICT_E_INVALID,
                "evict_kv_commit_stack_paged: page_size=%d must be a power of two in [1, 65536]", page_size);
  EVICT_REQUIRE(n_pages >= 1 && table_stride >= 1, EVICT_E_INVALID, "evict_kv_commit_stack_paged: n_pages=%d table_stride=%d",
                n_pages, table_stride);
  int shift = 0;
  while ((1 << shift) < page_size) ++shift;
  return kv_commit_impl("evict_kv_commit_stack_paged", ctx, dtype, Hkv, D, k_new, v_new, n_layers, tree_off, path, path_stride,
                        path_len, k_pools, v_pools, page_stride, kv_head_stride, ctx_len, capacity, ctx_len_out, B, stream,
                        KvPaging{block_table, table_stride, shift, n_pages});
}

}  // extern "C"
