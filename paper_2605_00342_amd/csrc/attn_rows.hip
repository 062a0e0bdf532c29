// Attention of the draft nodes for many query rows (bf16): kernel and launcher.
#include "device_utils.h"
#include "layer_launch.h"

#include <type_traits>

namespace evict {

// ------------------------------------------------------------------------------------
// bf16 tree-masked attention (head dimension 128) with 32 query rows per wavefront, four wavefronts per workgroup. The 16-row kernel
// (attn_partial_mfma_kernel) is bound by its LDS: every wavefront reads a whole chunk of keys and values for 16 rows, and V is
// transposed by 4-byte writes. Here
//  - both products run on the 32 x 32 x 16 MFMA with the query row in the lane (S^T = K Q^T, O^T = V^T P^T): a fragment read from
//    LDS feeds twice the matrix work, the softmax state of a row is the lane's own, and P goes from the accumulators of the
//    first product into the second without a move, since both take a block's keys in the same order;
//  - keys and values go from global memory straight into LDS, row-major (16-byte pieces XORed by their row against bank
//    conflicts); the V^T operand is read with the transposing LDS load;
//  - two buffers of 64 keys, the next chunk on its way during the work on this one, one barrier per chunk; 64 KiB, so two
//    workgroups per CU, whose matrix, vector and load phases overlap;
//  - the draft nodes are the last chunks of a sequence's last split instead of a split of their own: fewer partial rows;
//  - a batch is cut into equal shares by the kernel itself, which alone knows the sequences' lengths.
// (us, attention alone, 16 rows -> 32: 16 trees of 48 to 64 nodes, 32 heads on 4, contexts of 1024 to 2048 92 -> 40, 0.25 -> 0.57
// PFLOP/s; 4 such trees, contexts to 5555 48 -> 33; 128 nodes, context 4096 24 -> 21; 16 trees of 16 nodes, contexts to 6000 138 -> 38.)
// What bounds it now: a chunk of 64 keys takes a wavefront 1024 cycles of MFMA and 1200 (4 x 64 nodes, contexts to 5555) to 1500 (16 x 64, to 2048) of
// the vector unit, and two wavefronts per SIMD some 3000 for one each, as their phases overlap in part only; and some 9 us besides: the launch, 1.5 to 2.4 for the
// plan, 2.3 until the first chunk and the query rows are there, 1 to 3 for the partial rows. Tried: eight wavefronts that share a chunk, four
// buffers, three chunks on their way (6 % longer; the end of all workgroups at once costs more), loads sent between
// the first products instead of before them (30 % longer).
// ------------------------------------------------------------------------------------
constexpr int kRowsKeys = kAttnRowsKeys, kRowsPerWg = kAttnRowsPerWg, kRowsWaves = kRowsPerWg / 32;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) short s16x4;

__device__ __forceinline__ f32x16 mfma_32x32(u32x4 a, u32x4 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
// 4 keys of the lane's column: 16 lanes read 4 rows of 32 bytes and hand each lane one column
__device__ __forceinline__ uint2 lds_read_tr(const uint16_t* p) {
  return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)p));
}

// Sum over the lanes up to this one.
__device__ __forceinline__ int wave_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);  // row_shr 1, 2, 4, 8
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);  // row_bcast 15, 31
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);
  return v;
}

// PAGED: 0 contiguous caches, 1 pages of at least 4 positions, 2 smaller ones
template <int PAGED>
__global__ __launch_bounds__(kRowsWaves * 64) __attribute__((amdgpu_waves_per_eu(2))) void attn_rows_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ kc, const uint16_t* __restrict__ vc,
    long long seq_stride, long long head_stride, const int32_t* __restrict__ ctx_len, int max_ctx,
    const int32_t* __restrict__ tree_off, const uint16_t* __restrict__ k_new, const uint16_t* __restrict__ v_new,
    const uint64_t* __restrict__ anc, int Hq, int Hkv, int head_wgs, int chunks_per_split, int row_blocks, int T, float* __restrict__ part_o,
    float* __restrict__ part_ml, int32_t* __restrict__ row_splits, int n_single, int n_seq, const KvPaging pg,
    int32_t* __restrict__ status) {
  constexpr int D = 128, CH = D / 8, KB = D / 16, DT = D / 32;
  constexpr int KT = kRowsKeys / 32;                  // 32-key tiles of a chunk
  constexpr int LI = kRowsKeys * CH / 64 / kRowsWaves;  // 1 KiB wavefront loads of K (and of V) per wavefront
  // (objects of their own, so that the compiler can tell a read of one from a load into another in flight)
  __shared__ __attribute__((aligned(1024))) uint16_t s_b0[2 * kRowsKeys * D], s_b1[2 * kRowsKeys * D];  // K, V
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int G = Hq / Hkv;
  const int xcd = blockIdx.x & 7, id = blockIdx.x >> 3;
  int cps = chunks_per_split, split, g, b = 0, rb, splits, lo = 0, n, L, c_end;
  if (n_seq == 1) {
    // One tree: splits of a length the host chose. The row blocks of a unit (split, KV head) are on one XCD, whose L2 then fetches the
    // unit's keys once, and follow each other, but all first row blocks come first where most others may be empty (row_blocks < 0).
    n = n_single > 0 ? n_single : tree_off[1] - (lo = tree_off[0]);
    n = n > EVICT_MAX_TREE_NODES ? EVICT_MAX_TREE_NODES : n;
    L = ctx_len[0];
    L = L < 0 ? 0 : (L > max_ctx ? max_ctx : L);
    c_end = (L + kRowsKeys - 1) / kRowsKeys + (n + kRowsKeys - 1) / kRowsKeys;
    splits = head_wgs;
    const int rbs = row_blocks < 0 ? -row_blocks : row_blocks, units8 = (splits * Hkv + 7) >> 3;
    rb = row_blocks < 0 ? id / units8 : id % rbs;
    const int u = ((row_blocks < 0 ? id % units8 : id / rbs) << 3) + xcd;
    split = u / Hkv;
    g = u - split * Hkv;
    if (split >= splits || rb * kRowsPerWg >= n * G) return;
  } else {
    // A batch: the plan, by every wavefront for itself, a sequence per lane. A sequence's chunks (cache, then draft nodes) are cut into
    // splits of about `cps` chunks, the fewest that leave at most head_wgs workgroups per KV head (the host sees to it that one
    // split per sequence and row block is within that).
    int seq_n = 0, seq_chunks = 0, seq_lo = 0, seq_ctx = 0;
    if (lane < n_seq) {
      seq_lo = tree_off[lane];
      seq_n = tree_off[lane + 1] - seq_lo;
      seq_n = seq_n < 0 ? 0 : (seq_n > EVICT_MAX_TREE_NODES ? EVICT_MAX_TREE_NODES : seq_n);
      seq_ctx = ctx_len[lane];
      seq_ctx = seq_ctx < 0 ? 0 : (seq_ctx > max_ctx ? max_ctx : seq_ctx);
      seq_chunks = (seq_ctx + kRowsKeys - 1) / kRowsKeys + (seq_n + kRowsKeys - 1) / kRowsKeys;
    }
    const int seq_rbs = (seq_n * G + kRowsPerWg - 1) / kRowsPerWg;
    const int work = __builtin_amdgcn_readlane(wave_scan(seq_rbs * seq_chunks), 63);
    const int fewest = (work + head_wgs - 1) / head_wgs;
    cps = cps > fewest ? cps : fewest;
    int seq_splits = 0;
    for (;; cps += 1 + (cps >> 4)) {
      seq_splits = seq_rbs > 0 ? (seq_chunks + cps - 1) / cps : 0;
      if (__builtin_amdgcn_readlane(wave_scan(seq_rbs * seq_splits), 63) <= head_wgs || !__builtin_amdgcn_ballot_w64(seq_splits > 1)) break;
    }
    // Units (sequence, split, KV head) are dealt out to the 8 XCDs, one of every eight to each, by one further in the next eight, so
    // that no XCD gets all first or all last splits, and their row blocks follow each other. Only what has rows is counted: the
    // workgroups without work are the last ids (the dispatcher gives consecutive ids to the shader engines in turn whether or not
    // they have work: with empty row blocks between the others half of the CUs had none).
    const int seq_end = wave_scan(seq_splits) * Hkv, seq_begin = seq_end - seq_splits * Hkv;
    auto units_before = [&](int q) { return (q >> 3) + (((xcd - (q >> 3)) & 7) < (q & 7) ? 1 : 0); };
    const int mine = (units_before(seq_end) - units_before(seq_begin)) * seq_rbs;
    const int upto = wave_scan(mine);
    const uint64_t later = __builtin_amdgcn_ballot_w64(upto > id);
    if (!later) return;
    b = __builtin_ctzll(later);
    const int rbs = __builtin_amdgcn_readlane(seq_rbs, b), u0 = __builtin_amdgcn_readlane(seq_begin, b);
    const int in_seq = id - (__builtin_amdgcn_readlane(upto, b) - __builtin_amdgcn_readlane(mine, b));
    const int row8 = units_before(u0) + in_seq / rbs, u = 8 * row8 + ((xcd - row8) & 7) - u0;
    rb = in_seq % rbs;
    split = u / Hkv;
    g = u - split * Hkv;
    splits = __builtin_amdgcn_readlane(seq_splits, b);
    lo = __builtin_amdgcn_readlane(seq_lo, b);
    n = __builtin_amdgcn_readlane(seq_n, b);
    L = __builtin_amdgcn_readlane(seq_ctx, b);
    c_end = __builtin_amdgcn_readlane(seq_chunks, b);
    cps = (c_end + splits - 1) / splits;
  }
  const int R = n * G;
  // this split's chunks: n_ctx of the cache from key_begin on, then draft nodes
  const int c_begin = split * cps, c_all = (L + kRowsKeys - 1) / kRowsKeys;
  const int n_all = c_end - c_begin < cps ? c_end - c_begin : cps;  // (may be none: a context shorter than the host's bound)
  const int n_ctx = c_all - c_begin < 0 ? 0 : (c_all - c_begin < n_all ? c_all - c_begin : n_all);
  const int key_begin = c_begin * kRowsKeys;
  int key_end = key_begin + n_ctx * kRowsKeys;
  key_end = key_end > L ? L : key_end;
  const int tree_begin = c_begin + n_ctx - c_all;  // chunk of the draft nodes
  const int h = lane >> 5, ln = lane & 31;
  const int r0 = (rb * kRowsWaves + w) * 32;
  const bool active = r0 < R;
  const int rr = r0 + ln;
  const int r = rr < R ? rr : R - 1;
  const int qi = r / G, qh = r - qi * G;
  const int t = lo + qi;
  const size_t prow = ((size_t)split * T + t) * Hq + g * G + qh;

  if (n_all <= 0) {
    if (rr < R && h == 0) {  // nothing for the merge
      part_ml[prow * 2] = -INFINITY;
      part_ml[prow * 2 + 1] = 0.0f;
    }
    return;
  }

  u32x4 Qf[KB];
  uint64_t a0 = 0, a1 = 0;
  {
    const uint16_t* qrow = q + ((size_t)t * Hq + g * G + qh) * D + h * 8;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) Qf[kb] = *reinterpret_cast<const u32x4*>(qrow + kb * 16);
    if (n_all > n_ctx) { a0 = anc[2 * (size_t)t]; a1 = anc[2 * (size_t)t + 1]; }
  }
  const uint16_t* kctx = kc + (PAGED ? 0 : (size_t)b * seq_stride) + (size_t)g * head_stride;
  const uint16_t* vctx = vc + (PAGED ? 0 : (size_t)b * seq_stride) + (size_t)g * head_stride;
  // from the caches to the draft nodes' rows, in bytes (an offset: a choice between two pointers is turned into one between the
  // addresses of the lambdas' copies of them, which then live in scratch memory)
  const uintptr_t k_to_tree = (uintptr_t)(k_new + ((size_t)lo * Hkv + g) * D) - (uintptr_t)kctx;
  const int past_ctx = n - key_end;  // (likewise)
  const uintptr_t v_to_tree = (uintptr_t)(v_new + ((size_t)lo * Hkv + g) * D) - (uintptr_t)vctx;
  const int32_t* ptab = PAGED ? pg.table + (size_t)b * pg.table_stride : nullptr;
  const int pmask = (1 << pg.page_shift) - 1;

  // A wavefront-wide load brings 4 rows of 16 pieces; piece p of row `row` lies at p ^ (row & 15) of the row in K, where 16 lanes read
  // 16 bytes of a row each, and at p ^ 4 * (row & 3) in V, where 32 lanes read 64 bytes of 4 rows: the LDS serves 256 bytes per clock
  // to so many lanes, and none of them meet in a bank (conflict counter: 0; by row & 7 and 2 * (row & 7) half of the cycles).
  // Buffer loads: after global ones in flight the compiler waits for LDS reads by emptying their queue.
  const int srow = w * (4 * LI) + (lane >> 4), sp = lane & 15;
  // Pages of the 4-row groups of chunks c .. c + 3, one per lane (rows past the end: the last key's). Requested four chunks before
  // they are used: the counter is in order, and a wait for them would be one for every load of keys sent before.
  auto fetch_pages = [&](int c) __attribute__((always_inline)) -> int32_t {
    if (PAGED != 1 || n_ctx == 0) return 0;
    const int key = key_begin + c * kRowsKeys + lane * 4;
    return ptab[(key < key_end ? key : key_end - 1) >> pg.page_shift];
  };
  auto check_page = [&](int32_t page) __attribute__((always_inline)) -> int32_t {
    if (PAGED == 0 || (unsigned)page < (unsigned)pg.n_pages) return page;
    atomicOr(status, ST_BAD_PAGE);
    return 0;
  };
  // this wavefront's loads number `it` of K and V of chunk i; pages: of its 4-row groups, from lane `at_lane` on
  auto stage = [&](int i, int it, uint16_t* buf, int32_t pages, int at_lane) __attribute__((always_inline)) {
    const bool tree = i >= n_ctx;
    const int first = tree ? (tree_begin + i - n_ctx) * kRowsKeys : key_begin + i * kRowsKeys;
    const int most = key_end + (tree ? past_ctx : 0) - first - 1;  // rows past the end: of K the last one again, whose scores are masked; of V zeros, as a
                                                                   // weight of zero does not take an infinity out of the product
    const size_t step = tree ? (size_t)Hkv * D : (size_t)D;
    const uint16_t* kl = (const uint16_t*)((uintptr_t)kctx + (tree ? k_to_tree : 0)) + (PAGED && !tree ? 0 : (size_t)first * step);
    const uint16_t* vl = (const uint16_t*)((uintptr_t)vctx + (tree ? v_to_tree : 0)) + (PAGED && !tree ? 0 : (size_t)first * step);
    int row = srow + 4 * it;
    const int kp = sp ^ (row & 15), vp = sp ^ ((row & 3) << 2);
    const bool there = row <= most;
    row = there ? row : most;
    uint16_t *sk = buf + (w * LI + it) * 512, *sv = sk + kRowsKeys * D;
    if (PAGED == 2 && !tree) {  // a page of its own for every row, anywhere in the pool
      const int32_t page = check_page(ptab[(first + row) >> pg.page_shift]);
      const size_t off = (size_t)page * seq_stride + (size_t)((first + row) & pmask) * D;
      __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1)))*)(kl + off + kp * 8), (void __attribute__((address_space(3)))*)sk, 16, 0, 0);
      if (there) __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1)))*)(vl + off + vp * 8), (void __attribute__((address_space(3)))*)sv, 16, 0, 0);
      return;
    }
    if (PAGED == 1 && !tree) {  // the load's four rows are in one page (of at least 4 positions; those past the end read one and the same row)
      const int row0 = w * (4 * LI) + 4 * it < most ? w * (4 * LI) + 4 * it : most;
      const size_t off = (size_t)__builtin_amdgcn_readlane(pages, at_lane + w * LI + it) * seq_stride + (size_t)((first + row0) & pmask) * D;
      kl += off;
      vl += off;
      row -= row0;
    }
    const unsigned at = __umul24(row, (unsigned)step * 2);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc((void*)kl, 0, 0x7FFFFFFF, 0x27000),
                                             (void __attribute__((address_space(3)))*)sk, 16, at + kp * 16, 0, 0, 0);
    if (there)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc((void*)vl, 0, 0x7FFFFFFF, 0x27000),
                                               (void __attribute__((address_space(3)))*)sv, 16, at + vp * 16, 0, 0, 0);
  };
  auto stage_all = [&](int i, uint16_t* buf, int32_t pages, int at_lane) __attribute__((always_inline)) {
    // (before the chunk's loads: a write behind one that is on its way into the same object would wait for it)
    const int past = i >= n_ctx ? n - (tree_begin + i - n_ctx) * kRowsKeys : key_end - key_begin - i * kRowsKeys;
    if (past < kRowsKeys) {
#pragma unroll
      for (int it = 0; it < LI; ++it)
        if (srow + 4 * it >= past) *reinterpret_cast<u32x4*>(buf + kRowsKeys * D + (w * LI + it) * 512 + lane * 8) = u32x4{0, 0, 0, 0};
    }
#pragma unroll
    for (int it = 0; it < LI; ++it) stage(i, it, buf, pages, at_lane);
  };

  f32x16 O[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) O[dt] = f32x16{0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  float lsum = 0.0f;         // of this lane's keys: half of every tile's
  float m_run = -INFINITY;   // running maximum of the scaled scores
  const float scale = 1.0f / sqrtf((float)D);
  const float c2 = scale * 1.44269504088896341f;

  // V^T fragment j (key group j / DT, output tile j % DT): lane = output column, keys 16 * kg + 4 * h + {0..3} and 8 more
  const int vrow = 4 * h + ((lane & 15) >> 2);
  const int vpart = vrow * D + (lane & 1) * 4;
  const int vcol = (((lane >> 4) & 1) * 2 + ((lane & 3) >> 1)) ^ ((vrow & 3) << 2);  // piece of the 16 columns' 32 bytes
  const int kcol = h ^ (ln & 15);
  auto compute = [&](auto full_tag, uint64_t vis, const uint16_t* sk) __attribute__((always_inline)) {
    constexpr bool full = decltype(full_tag)::value;
    const uint16_t* sv = sk + kRowsKeys * D;
    auto load_k = [&](u32x4(&f)[KT], int kb) __attribute__((always_inline)) {
#pragma unroll
      for (int kt = 0; kt < KT; ++kt) f[kt] = *reinterpret_cast<const u32x4*>(sk + (kt * 32 + ln) * D + ((kcol ^ (kb * 2)) << 3));
    };
    auto load_v = [&](u32x4& f, int j) __attribute__((always_inline)) {
      const uint16_t* at = sv + (j / DT) * 16 * D + vpart + ((vcol ^ (j % DT * 4)) << 3);
      const uint2 x = lds_read_tr(at), y = lds_read_tr(at + 8 * D);  // (rows 8 apart have the same XOR)
      f = u32x4{x.x, x.y, y.x, y.y};
    };
    // Fragments are requested kAheadK / kAheadV products before they are used; the fences keep the compiler from moving the
    // requests to their uses.
    constexpr int kAheadK = 2, kAheadV = 4, NV = KT * 2 * DT;
    f32x16 S[KT];
    u32x4 kf[kAheadK + 1][KT], vf[kAheadV + 2];
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) S[kt] = f32x16{0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int kb = 0; kb < kAheadK; ++kb) load_k(kf[kb], kb);
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
      if (kb + kAheadK < KB) load_k(kf[(kb + kAheadK) % (kAheadK + 1)], kb + kAheadK);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int kt = 0; kt < KT; ++kt) S[kt] = mfma_32x32(kf[kb % (kAheadK + 1)][kt], Qf[kb], S[kt]);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int j = 0; j < kAheadV; ++j) load_v(vf[j], j);
    __builtin_amdgcn_sched_barrier(0);
    // lane: keys kt * 32 + 8 * (e / 4) + 4 * h + e % 4 of its row
    float mx = -INFINITY;
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
      if (!full) {
        const uint32_t v32 = (uint32_t)(vis >> (kt * 32)) >> (4 * h);
#pragma unroll
        for (int e = 0; e < 16; ++e) S[kt][e] = (v32 >> (8 * (e >> 2) + (e & 3))) & 1u ? S[kt][e] : -INFINITY;
      }
#pragma unroll
      for (int e = 0; e < 16; e += 2) mx = fmaxf(fmaxf(S[kt][e], S[kt][e + 1]), mx);
    }
    {
      const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_int(mx), __float_as_int(mx), false, false);
      mx = fmaxf(__int_as_float(sw[0]), __int_as_float(sw[1]));
    }
    // The maximum is that of all keys so far: the largest weight of a row is then exactly 1 in bf16, not rounded, which counts where a
    // few keys have most of the weight. (Moved only when outgrown by e^5, it saved most rescalings, 4 x 64 nodes, contexts to 5555, 2 us,
    // and the output was off from 64-bit sums by 1.17 times the 16-row kernel's error at scores of deviation 2.4; this way 0.99.)
    const float m_new = mx * scale;
    if (__builtin_amdgcn_ballot_w64(m_new > m_run)) {
      const float m_up = fmaxf(m_run, m_new);
      const float alpha = m_run == -INFINITY ? 0.0f : __expf(m_run - m_up);
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) O[dt] *= alpha;
      lsum *= alpha;
      m_run = m_up;
    }
    // exp(s * scale - m) = 2^(s * c2 + moff); a row without a visible key so far has m = -inf and gets zeros
    const float moff = !full && m_run == -INFINITY ? 0.0f : -m_run * 1.44269504088896341f;
    u32x4 P[KT * 2];
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
      for (int e = 0; e < 16; e += 2) {
        const float p0 = __builtin_amdgcn_exp2f(fmaf(S[kt][e], c2, moff)), p1 = __builtin_amdgcn_exp2f(fmaf(S[kt][e + 1], c2, moff));
        const uint32_t pk = pack_bf16x2(p0, p1);
        P[kt * 2 + (e >> 3)][(e & 7) >> 1] = pk;
        lsum = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, pk), __builtin_bit_cast(bf16x2_t, 0x3F803F80u), lsum, false);  // of the rounded weights
      }
#pragma unroll
    for (int j = 0; j < NV; j += 2) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
        if (j + i + kAheadV < NV) load_v(vf[(j + i + kAheadV) % (kAheadV + 2)], j + i + kAheadV);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < 2; ++i) O[(j + i) % DT] = mfma_32x32(vf[(j + i) % (kAheadV + 2)], P[(j + i) / DT], O[(j + i) % DT]);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // Chunk i lies in buffer i % 2, chunk i + 1 is on its way during the work on it. A wavefront waits for its own loads, then for
  // everybody's at the barrier, which also says that all have left the other buffer.
  auto chunk_barrier = [&]() __attribute__((always_inline)) {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(7 << 4);  // vmcnt(0), lgkmcnt(0): by the builtin, so that the compiler does not wait for them again
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  int32_t p_now = fetch_pages(0), p_next = fetch_pages(4);
  p_now = check_page(p_now);
  auto turn_pages = [&](int c) __attribute__((always_inline)) {  // before chunk c is requested
    if (PAGED == 1 && (c & 3) == 0) {
      p_now = check_page(p_next);
      p_next = fetch_pages(c + 4);
    }
  };
  auto step_full = [&](int i, uint16_t* buf, uint16_t* ahead) __attribute__((always_inline)) {
    chunk_barrier();
    turn_pages(i + 1);
    if (i + 1 < n_all) stage_all(i + 1, ahead, p_now, ((i + 1) & 3) * 16);
    if (active) compute(std::true_type{}, 0, buf);
  };
  const int n_full = n_ctx > 0 ? (key_end - key_begin) / kRowsKeys : 0;  // chunks without a mask
  stage_all(0, s_b0, p_now, 0);
  int i = 0;
  for (; i + 1 < n_full; i += 2) {
    step_full(i, s_b0, s_b1);
    step_full(i + 1, s_b1, s_b0);
  }
  // the last chunk of an odd count, the ragged last chunk of the cache, the draft nodes
  for (; i < n_all; ++i) {
    chunk_barrier();
    turn_pages(i + 1);
    uint16_t *buf = i & 1 ? s_b1 : s_b0, *ahead = i & 1 ? s_b0 : s_b1;
    if (i + 1 < n_all) stage_all(i + 1, ahead, p_now, ((i + 1) & 3) * 16);
    if (!active) continue;
    const bool tree = i >= n_ctx;
    const int part = tree_begin + i - n_ctx;
    const int left = tree ? n - part * kRowsKeys : key_end - key_begin - i * kRowsKeys;
    const uint64_t there = left >= 64 ? ~0ull : (1ull << left) - 1ull;
    compute(std::false_type{}, tree ? (part == 0 ? a0 : a1) & there : there, buf);
  }
  if (!active) return;
  {
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_int(lsum), __float_as_int(lsum), false, false);
    lsum = __int_as_float(sw[0]) + __int_as_float(sw[1]);
  }
  if (rr >= R) return;
  if (h == 0) {
    part_ml[prow * 2] = m_run;
    part_ml[prow * 2 + 1] = lsum;
    if (n_seq > 1 && split == 0 && g == 0 && qh == 0) row_splits[t] = splits;
  }
  float* dst = part_o + prow * D + 4 * h;
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int e = 0; e < 16; e += 4)
      *reinterpret_cast<f32x4*>(dst + dt * 32 + 2 * e) = f32x4{O[dt][e], O[dt][e + 1], O[dt][e + 2], O[dt][e + 3]};
}

int launch_attn_rows(const evict_ctx* c, const void* kc, const void* vc, long long seq_stride, long long head_stride, const int32_t* ctx_len,
                     int max_ctx_host, const int32_t* tree_off, int B, int T, const void* k_new, const void* v_new, int* nsplits, hipStream_t s) {
  const evict_model_desc& m = c->m;
  const int G = m.Hq / m.Hkv;
  const int max_nodes = T < EVICT_MAX_TREE_NODES ? T : EVICT_MAX_TREE_NODES;
  const int max_rb = (max_nodes * G + kRowsPerWg - 1) / kRowsPerWg;
  const int chunks = (max_ctx_host + kRowsKeys - 1) / kRowsKeys + (max_nodes + kRowsKeys - 1) / kRowsKeys;
  const int target = attn_rows_wgs(B, T, m.Hq, m.Hkv, max_ctx_host);
  int cps = (chunks + kAttnRowsMaxSplits - 1) / kAttnRowsMaxSplits, head_wgs, row_blocks = max_rb;
  dim3 grid;
  if (B == 1) {
    const int want = attn_rows_splits(target, m.Hkv, max_rb);
    cps = cps > (chunks + want - 1) / want ? cps : (chunks + want - 1) / want;
    head_wgs = *nsplits = (chunks + cps - 1) / cps;
    if (c->t_dev) row_blocks = -max_rb;
    grid = dim3((head_wgs * m.Hkv + 7) / 8 * 8 * max_rb);
  } else {
    const int max_rbs = T * G / kRowsPerWg + B;  // row blocks of all sequences
    head_wgs = target / m.Hkv > max_rbs ? target / m.Hkv : max_rbs;
    *nsplits = (chunks + cps - 1) / cps;  // at most
    // (a unit's row blocks are on one XCD: one XCD may have a unit more than another of every sequence)
    grid = dim3((head_wgs * m.Hkv / 8 + B * max_rb + 1) * 8);
  }
#define EVICT_ATTN_ROWS(PAGED_)                                                                                                      \
  hipLaunchKernelGGL(attn_rows_kernel<PAGED_>, grid, dim3(kRowsWaves * 64), 0, s, (const uint16_t*)c->q, (const uint16_t*)kc,        \
                     (const uint16_t*)vc, seq_stride, head_stride, ctx_len, max_ctx_host, tree_off, (const uint16_t*)k_new,          \
                     (const uint16_t*)v_new, c->anc, m.Hq, m.Hkv, head_wgs, cps, row_blocks, T, c->part_o, c->part_ml, c->row_splits,    \
                     (B == 1 && !c->t_dev) ? T : 0, B, c->paging, c->status)
  if (!c->paging.table) EVICT_ATTN_ROWS(0);
  else if (c->paging.page_shift >= 2) EVICT_ATTN_ROWS(1);
  else EVICT_ATTN_ROWS(2);
#undef EVICT_ATTN_ROWS
  return launch_status("attn_rows_kernel");
}

}  // namespace evict
