// Which kernel a call takes where several are built for it: rules on sizes and on the launch-shape knobs of a context
// (evict_tune), without any device code, so that they can be checked on the host.
#pragma once

namespace evict {

// Knobs of the expert GEMMs. A knob that was set asks for the kernels it describes, so the tiled kernels, which have none
// of these choices, are left out: weights by ordinary loads, operand staging, refill order, units per workgroup, tiles.
// (Non-temporal loads are what the tiled kernels use, so nt_loads = 1 leaves them in.)
struct MoeKnobs {
  int nt, gateup_kernel, down_kernel, pair_down, down_ws, nt_loads, lds_dma, prefetch, chunk_gateup, chunk_down;
};
inline bool moe_knobs_auto(const MoeKnobs& k) {
  return k.nt == 0 && k.gateup_kernel == 2 && k.down_kernel == 1 && k.pair_down == 2 && k.down_ws == 0 && k.nt_loads != 0 &&
         k.lds_dma == 1 && k.prefetch == 1 && k.chunk_gateup == 0 && k.chunk_down == 0;
}

// The tiled expert kernels (bf16, knobs as above, shapes that are built) for T tokens of k experts out of E; the gate/up
// projection has nkb contraction blocks and `pairs` strip pairs; strip: the call would else take the strip kernels.
// They take up to 96 tokens of an expert through one weight stream where the other kernels take 16 (or 32) at a time, but
// their workgroups run longer. They pay once
//  - experts mostly have several token tiles. Whole layers (us, before -> tiled): 128 experts 96 nodes 143 -> 131, 175 -> 173,
//    217 -> 211 (child noise 0.2, 0.5, 1.0) but 64 nodes 115 -> 110, 149 -> 148, 180 -> 183; a rank's share of 128 experts
//    128 nodes 175 -> 150, 4 x 100 nodes 309 -> 212. So from an average of 6 tokens per expert; 8 where six wavefronts do not
//    share out an expert's strip pairs evenly (width 1408: 64 nodes, 6 tokens per expert, 2 % faster to 2 % slower by the
//    routing; 86 nodes, 8 tokens, 170 -> 150, 223 -> 192, 255 -> 233); 10 over 4096 columns, where the contraction-split
//    kernel keeps its token operand;
//  - the experts' chunks of six strip pairs can fill the 256 CUs. 16 experts of width 256 are 48 workgroups: gate/up of 96
//    nodes 17 -> 28 us; of width 768, 128 workgroups, 26 -> 30.
// Over 2048 columns their sums are one chain, as those of the strip kernels, where the contraction split has eight: they stand
// in for the strip kernels only.
constexpr bool experts_tiled(int T, int k, int E, int nkb, int pairs, bool strip) {
  if (nkb <= 64 && !strip) return false;
  if (E * ((pairs + 5) / 6) < 256) return false;
  return T * k >= (nkb <= 64 ? (pairs % 6 == 0 ? 6 : 8) : 10) * E;
}

// Knobs of the QKV / output projections, likewise.
inline bool dense_knobs_auto(int kernel, int nt, int ntw, int units, int nt_loads) {
  return kernel == 2 && nt == 0 && ntw == 0 && units == 0 && nt_loads != 0;
}

// Workgroups of a tiled projection that takes `strips` of the n_strips strips and one of the token groups each. Ids go
// round-robin over the 8 XCDs, a strip group's token groups on one XCD, so the strip groups are padded to a multiple of 8 and
// the XCDs with one group more decide: 20 strip groups x 12 token groups are 36 workgroups for each of four XCDs of 32 CUs
// and not one round (160 strips of 64 blocks, 370 tokens: 28 us, and 20 with the next larger tile).
constexpr int tile_grid(int n_strips, int strips, int token_groups) {
  return ((n_strips + strips - 1) / strips + 7) / 8 * 8 * token_groups;
}

// The LM head (bf16, auto knobs, shapes that are built): the tiled kernel for T tokens, n_strips 16-row strips and nkb
// contraction blocks. It reads the weights once for up to 96 tokens, but a workgroup takes 8 or 16 strips, so it needs many.
// 151936 rows (us, contraction split -> tiled). 64 blocks: 16 tokens 101 (not yet: 112), 32 tokens 116 (118), 48 tokens
// 161 -> 124, 64 173 -> 129, 96 211 -> 135, 128 313 -> 171. 128 blocks, where the split kernel re-reads its token operand for
// every strip: 9 tokens 209 (214), 12 229 -> 215, 16 254 -> 216, 33 690 -> 224, 64 743 -> 244, 128 1345 -> 323.
// 64 blocks, 96 tokens: 32000 rows 46 -> 44, but 16000 rows 37 (43), 4096 rows 25 (40). 128 blocks: 16000 rows 16 tokens
// 38 -> 35, but 8192 rows 26 (32); from 17 tokens on the tiled kernel is the better at 1024 rows already, 61 -> 30.
constexpr bool lm_tiled(int T, int n_strips, int nkb) {
  if (n_strips % 2 != 0) return false;
  return (nkb == 64 && T > 32 && n_strips > 1024) || (nkb == 128 && (T > 16 || (T >= 12 && n_strips > 768)));
}

// Strips per workgroup of the contraction split for the LM head: 8 from 17 tokens on; for one token tile 2, but 8 from 13
// tokens on if that leaves about a workgroup per CU. (64 blocks, 2 strips -> 8, us: 151936 rows 16 tokens 121 -> 111, 9 tokens
// 109 -> 109; 32000 rows 16 tokens 33.7 -> 31.1; 102400 rows 12 tokens 81 -> 84, 9 tokens 76 -> 83; 16000 rows 16 tokens
// 24.1 -> 24.8.)
constexpr int lm_units(int T, int n_strips) { return T > 16 || (T > 12 && n_strips > 1024) ? 8 : 2; }

// With two token tiles a workgroup fills a CU, so the strips can be dealt out in one round of 256 workgroups instead of 8 at a
// time, whose last round may be partly empty and whose every workgroup fetches the token operand.
constexpr int lm_strips(int T, int n_strips) {
  const int units = lm_units(T, n_strips), round = (n_strips + 255) / 256;
  return T > 16 && round > units ? round : units;
}

// Where that pays: bf16, strips of up to 64 blocks, and not with so much for each workgroup that the last ones to end cost more
// than is saved: 2048 blocks, from 25 tokens on, whose operand is the larger, 2432. (T of 17 .. 32, arg max and score rows, time
// against 8 strips each: 2560 strips of 32 blocks 0.79 .. 0.82, 9496 of 32 0.88 .. 0.96, 9496 of 48 0.95 .. 1.00, 6400 of 64 0.94 .. 0.98,
// 8016 of 64 0.97 .. 1.03, most below 1, 3142 of 24 1.00 .. 1.03, 9496 of 64, the weights of three heads in turn, T up to 24
// 1.00 .. 1.02, 26 to 30 0.98 .. 1.00, 32 0.97 .. 0.99; but 8016 of 96 0.99 .. 1.06, 2049 and 4097 of 128 1.03 .. 1.07; 32-bit storage, 4096
// of 64, 0.98 .. 1.03.) Several groups of 32 tokens are no longer one round: only with short strips, whose workgroups are all
// start (33 to 128 tokens, 2560 to 15625 strips of 16 to 48 blocks 0.75 .. 1.01; 4097 of 64 0.94 .. 1.04).
constexpr bool lm_one_round(int T, int n_strips, int nkb, bool bf16) {
  return bf16 && nkb <= 64 && (n_strips + 255) / 256 * nkb <= (T > 24 ? 2432 : 2048) && (T <= 32 || nkb <= 48);
}

// Strips of 64 blocks in bf16, whose scores or candidates a workgroup keeps until its strips are done (gemm_stream_kernel), are dealt out in
// one round from 13 tokens on already (us, 8 strips each -> one round, score rows / arg max: 6400 strips, 16 tokens 74 / 75 -> 67 / 70; 9496, 16 tokens 106 / 102 ->
// 103 / 103, 17 tokens 109 / 105 -> 103 / 104, 24 tokens 114 / 105 -> 104 / 103). With one token tile two workgroups share a CU, but the round of 256 is the
// better (19 strips each 100 / 96; 12 tokens, two strips each, 97 / 98, one round 95 / 97). The line lies where the measurements of the form before ended. Past
// it, 32 tokens: 42 strips each 134 / 121 -> 118 / 115, 47 147 / 128 -> 132 / 129, 48 149 / 132 -> 141 / 136; 16 tokens: 47 132 / 125 -> 128 / 128, 48 135 / 128 -> 135 / 137.
constexpr int lm_deal(int T, int n_strips, int nkb, bool bf16) {
  const int round = (n_strips + 255) / 256;
  if (bf16 && nkb == 64 && T > 12 && T <= 32 && n_strips > 4096 && round * nkb <= 2432) return round;
  return lm_one_round(T, n_strips, nkb, bf16) ? lm_strips(T, n_strips) : lm_units(T, n_strips);
}

// Candidates of the arg max, one token tile, kept by a workgroup until its strips are done (ARGMAX_WG): from so many strips on that the fewer
// stores and candidates make up for the exchange at its end, which few strips per workgroup do not. (Head and arg max, us, strip by strip ->
// kept. 64 blocks, 16 tokens: 64 strips 13.0 -> 13.9, 500 15.4 -> 15.7, 1000 20.7 -> 20.9, 2000 32.1 -> 32.1, 3142 43.9 -> 42.3, 9496 109 -> 104; 24
// blocks: 500 12.9 -> 13.3, 1000 14.7 -> 15.0, 2000 20.8 -> 19.7, 9496 57 -> 49; 128 blocks, 8 tokens: 64 17.2 -> 17.7, 2000 49.5 -> 49.7, 3142 75.8 -> 75.3.)
constexpr bool lm_keeps_best(int n_strips, int nkb, bool bf16) {
  return bf16 && (nkb % 64 == 0 ? n_strips > 2048 : nkb == 24 && n_strips > 1536);
}

// Score rows kept in LDS until then (ROWS_WG). (us, strip by strip -> kept: 64 blocks, 32 tokens 500 strips 19.1 -> 18.9, 3142 43.3 -> 41.2, 9496
// 117 -> 106; 48 tokens 64 strips 13.8 -> 14.4, 1000 19.5 -> 19.6; 16 tokens 64 strips 9.8 -> 10.2, 3142 40.0 -> 40.0, 6400 79 -> 72; 8 tokens
// 9496 100.6 -> 99.9. 128 blocks, 8 tokens: 2000 46.0 -> 46.3, 9496 187.4 -> 187.9, 24 tokens 4097 106.4 -> 104.5.)
constexpr bool lm_keeps_rows(int T, int n_strips, int nkb, bool bf16) {
  return bf16 && nkb % 64 == 0 && n_strips > 2048 && (nkb == 64 || T > 12);
}

// TopK beside the union (up to 32 tokens): four tokens per wavefront, in rows of 16 lanes with room for a pick each, once some of
// the 16 wavefronts would have two tokens. (TopK and union, us, one -> four: 32 tokens 9.1 -> 7.3, one token 5.3 -> 6.6. Whole layers: 8 picks
// of 128 experts, 9 tokens 41.5 -> 42.1, 17 43.3 -> 43.3, 24 44.2 -> 43.8, 32 45.5 -> 44.1; 16 picks, 9 tokens 43.9 -> 44.8, 17 46.6 -> 46.9, 24
// 48.0 -> 47.5. With 16 scores in a lane instead of 8 the chain of a pick is longer: 8 of 256, 9 tokens 42.8 -> 44.2, 24 46.1 -> 46.7, 28
// 47.4 -> 46.9; 16 of 256 45.7 -> 49.3, 52.5 -> 54.1, 54.4 -> 54.4; 4 of 160, 24 tokens 43.7 -> 43.8, 28 44.7 -> 44.1.)
constexpr bool topk_by_rows(int T, int E, int k) { return k <= 16 && T >= (E > 128 ? 28 : 17); }

// bf16 attention with 32 query rows per wavefront (attn_rows_kernel) instead of 16 (attn_partial_mfma_kernel), for B trees of T nodes together
// and contexts of up to max_ctx positions. Its workgroups take 128 rows of a KV head and run through chunks of 64 keys.
constexpr int kAttnRowsKeys = 64, kAttnRowsPerWg = 128, kAttnRowsMaxSeqs = 64;
// Chunks of all row blocks, KV heads and sequences, by the longest context.
constexpr long long attn_rows_work(int B, int T, int Hq, int Hkv, int max_ctx) {
  const long long rbs = ((long long)T * (Hq / Hkv) + kAttnRowsPerWg - 1) / kAttnRowsPerWg;
  return (rbs > B ? rbs : B) * Hkv * ((max_ctx + kAttnRowsKeys - 1) / kAttnRowsKeys + 1);
}
// Attention and merge, us, 16 rows -> 32. Many chunks: 1 x 64 nodes of 4 KV heads of 8, ctx 6000 25.0 -> 22.3, 1 x 128 ctx 16000
// 70.3 -> 54, 4 x 64 ctx 6000 56.6 -> 40, 16 x 64 ctx 2048 101.5 -> 49; 16 heads of one, 4 x 64 ctx 600 19.4 -> 15. Many small trees, whose empty
// row blocks the 16-row kernel deals out between the others (half to three quarters of the CUs get none): 16 x 16 ctx 600 51.4 -> 18,
// 64 x 8 ctx 100 45.2 -> 23. One tree that fills at most two wavefronts, which then take a chunk of 64 keys each where the other kernel
// takes 128: 1 x 8 ctx 600 10.0 -> 9.0, 16 heads of one, 1 x 64 ctx 2048 16.2 -> 14.1.
// Not where few chunks leave most of a workgroup's time to its start and its end: 1 x 64 ctx 600 13.4 (14.9), 1 x 32 ctx 600 11.5 (13.0), one KV
// head, 2 x 128 ctx 600 12.8 (17.1), 1 x 64 ctx 6000 15.8 (16.7). The line lies higher where the 16-row kernel has few empty row blocks (whole
// small layers, us, 16 rows -> 32, chunks in brackets): one or two KV heads, 1 to 4 trees, 8/1 2 x 96 ctx 3000 58.0 -> 61.7 (576), 3 x 128 ctx 2048 65.0 -> 66.5
// (792), 16/2 1 x 64 ctx 4096 55.0 -> 56.4 (520), but 8/1 1 x 128 ctx 8000 62.2 -> 62.1 (1008), and with long contexts, where both cut as often as they
// may, 8/1 1 x 64 ctx 8192 51.7 -> 52.3 (516), 10000 54.6 -> 53.2 (632), a layer of 4096 columns, 1 x 44 ctx 15161 103.1 -> 101.2 (714); 64 heads on 8, 1 x 48 ctx 2048 65.7 -> 66.7 (792), 3000 69.6 ->
// 67.8 (1128); 2 to 4 trees of more than 72 nodes, 16/16 2 x 96 ctx 1000 69.3 -> 70.4 (544), 1500 71.2 -> 72.0 (800), 2048 76.1 -> 72.4 (1056). And where
// it has none, as a batch of trees of few rows lies within one of its workgroups (8 nodes of 4 trees, 16 heads of one: ctx 1000 47.4 -> 48.2,
// 3000 60.4 -> 61.4, 4096 67.2 -> 62.7; one node, 8 trees 1000 51.3 -> 55.1, 2048 62.1 -> 56.5): from 16 chunks a workgroup on, or with more units
// (sequences x KV heads) than half of the CUs from 8 on (12 trees of one node 300 47.0 -> 48.2, 600 58.0 -> 56.3), or more than CUs. One tree has to pass attn_rows_one_tree as well.
constexpr bool attn_rows_applies(int D, int B, int T, int Hq, int Hkv, int max_ctx) {
  if (D != 128 || B > kAttnRowsMaxSeqs) return false;
  const long long work = attn_rows_work(B, T, Hq, Hkv, max_ctx), units = (long long)B * Hkv, rows = (long long)T * (Hq / Hkv);
  if (rows <= 64) return B == 1 || work >= 16 * 256 || units > 256 || (units > 128 && work >= 5 * 256);
  if (B >= 16) return true;
  const bool few_empty = max_ctx <= 8192 && B <= 4 && (Hkv <= 2 || (B == 1 ? Hq >= 64 : T > 72 * B));
  return work >= (few_empty ? 830 : 400);
}
// One tree: only from 12 chunks per CU on, where it is clearly the faster. Below, it gains or loses a few percent of such a small layer, and another
// order of sums takes a token whose last expert is nearly tied to another expert, 4e-2 of its row, which a batch's many tokens average out and the few
// of one tree, or the score rows behind a stack of layers, do not. (Whole small layers, us, 16 rows -> 32, chunks in brackets. 4 heads of 8: 1 node ctx 2048
// 41.5 -> 41.4 (132), 16 nodes ctx 3000 50.6 -> 50.2 (192), 41 ctx 3000 60.7 -> 61.0 (576), 64 ctx 5000 67.0 -> 67.1 (1280), 128 ctx 5000 79.5 -> 81.4 (2560), 41 ctx 12000
// 69.8 -> 70.6 (2268), 64 ctx 8000 71.5 -> 69.9 (2016); 128 ctx 8000 89.5 -> 88.3 (4032), ctx 12000 103.5 -> 92.4 (6048), ctx 32000 171.8 -> 137.1, 41 ctx 20000 93.8 -> 79.1 (3768),
// 64 ctx 20000 89.1 -> 82.6. 16 heads of one: 64 ctx 8000 63.7 -> 63.9 (2016), 16 ctx 5000 56.5 -> 52.8 (1280), 64 ctx 20000 78.6 -> 75.6 (5024). One head of 8: 64 ctx 32000
// 73.4 -> 74.0 (2008), 128 ctx 32000 83.9 -> 81.9 (4016).)
constexpr bool attn_rows_one_tree(int T, int Hq, int Hkv, int max_ctx) { return attn_rows_work(1, T, Hq, Hkv, max_ctx) >= 12 * 256; }
// Its loads go straight into LDS, 16 bytes a lane, and so need rows of the caches at multiples of 16 bytes; caches at other strides, which the 16-row
// kernel reads through registers, stay there. (One sequence: the distance to the next is not used.)
constexpr bool attn_rows_strides(int B, long long seq_stride, long long head_stride) {
  return head_stride % 8 == 0 && (B == 1 || seq_stride % 8 == 0);
}
// Workgroups to cut the splits for: one per CU, or two, which overlap each other's phases but leave twice the partial rows to the
// merge, once they have 16 chunks and more (whole small layers, us, one per CU, two, chunks in brackets: 4 heads of 8, 4 x 64 nodes ctx 2048 75.1, 77.2 (2112),
// 1 x 128 ctx 6000 75.5, 78.2 (3040), 8 x 64 ctx 2048 110.2, 105.3 (4224), 16 x 64 156.5, 145.4 (8448); 16 heads of one, 8 x 8 ctx 2048 71.3, 61.7 (4224). It is not
// the chunks alone: 16 heads of one, 4 x 128 ctx 6000 117, 121 (6080), 16 x 8 ctx 600 72.1, 67.3 (2816); one head of 8, 8 x 128 ctx 6000 101, 110 (6080)).
constexpr int attn_rows_wgs(int B, int T, int Hq, int Hkv, int max_ctx) {
  return attn_rows_work(B, T, Hq, Hkv, max_ctx) >= 16 * 256 ? 512 : 256;
}
// One tree: most splits that this leaves for Hkv heads of `rbs` row blocks. A unit's row blocks are on one XCD, so what counts is the fullest
// XCD: 21 splits of 4 heads are 84 units, 11 of them on four XCDs, and with three row blocks each 33 workgroups on 32 CUs. (48 nodes of 4
// heads of 8, whole small layer, us, 21 splits by the total alone -> 18 and 19: ctx 8000 66.5 -> 62.6, ctx 12000 73.5 -> 65.5; the 16-row kernel 63.5 and 69.2.)
constexpr int attn_rows_splits(int wgs, int Hkv, int rbs) {
  const int units = wgs / 8 / rbs * 8;
  return units / Hkv > 1 ? units / Hkv : 1;
}

// Weight loads of the down projections, as the knob says; auto: non-temporal, but ordinary ones for the 8 contraction blocks
// of expert width 256 (13.8 us for 40 experts; the better from 64 tokens on).
inline int down_nt_loads(int knob, int nkb) { return knob == 2 ? (nkb == 8 ? 0 : 1) : knob; }

// Strip pairs per chunk of the contraction-split gate/up kernel over 4096 columns, for `slots` slots of the work list and
// `pairs` strip pairs per expert. A workgroup fills a CU, so what counts is how the slots * pairs / c chunks fall into rounds
// of 256: a full round streams at the rate of memory, 10 us per pair of a chunk; the last takes at least a chunk's own walk,
// 4 us per pair and 8 to start. (us for c = 1, 2, 3, 4, and the kernel with steps of 64 blocks that this one replaced; width
// 192: 43 slots 34.0, 37.7, 29.2, 32.4, old 35.5; 46 slots 34.2, 37.4, 27.7, 34.6, old 37.8; 17 slots 14.1, 17.9, 22.3,
// 26.3, old 16.0; 66 slots 42.0, 40.3, 49.6, 38.8, old 45.1. Width 256, c = 1, 2, 4: 35 slots 35.1, 37.6, 31.3, old 36.4;
// 130 slots 90.3, 91.5, 103.3, old 97.8. Always two is slower than the old kernel at 16 of
// ninety such points.) From two full rounds of two pairs on the rounds no longer decide but the operand traffic and, where experts
// have several slots, the weights that these find in L2: two pairs there (width 256, 4 x 80 nodes: 170 us, 183 by rounds; 2 x 100
// nodes 77, 90).
// Worked out on the device, with the slots, from the counts of chunks that the host has divided out.
struct ChunkCounts {
  int n[4];  // chunks of 1 .. 4 pairs an expert's pairs make, 0 where that does not divide them
};
constexpr ChunkCounts gateup_chunk_counts(int pairs) {
  ChunkCounts k = {};
  for (int c = 1; c <= 4; ++c) k.n[c - 1] = pairs % c == 0 ? pairs / c : 0;
  return k;
}
constexpr int gateup_chunk(int slots, const ChunkCounts& counts) {
  if (counts.n[1] > 0 && slots * counts.n[1] >= 512) return 2;
  int best = 1, best_cost = 0x7fffffff;
#pragma unroll
  for (int c = 1; c <= 4; ++c) {
    const int n = slots * counts.n[c - 1], rest = n & 255;
    const int walk = 4 * c + 8, share = 10 * c * rest >> 8;
    const int cost = (n >> 8) * 10 * c + (rest == 0 ? 0 : (walk > share ? walk : share));
    if (counts.n[c - 1] > 0 && cost < best_cost) { best_cost = cost; best = c; }
  }
  return best;
}

}  // namespace evict
