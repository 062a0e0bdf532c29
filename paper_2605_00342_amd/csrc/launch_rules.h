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

// Knobs of the QKV / output projections, likewise.
inline bool dense_knobs_auto(int kernel, int nt, int ntw, int units, int nt_loads) {
  return kernel == 2 && nt == 0 && ntw == 0 && units == 0 && nt_loads != 0;
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
// ninety such points.)
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
  int best = 1, best_cost = 0x7fffffff;
#pragma unroll
  for (int c = 1; c <= 4; ++c) {
    const int n = slots * counts.n[c - 1], rest = n & 255;
    const int walk = 4 * c + 8, share = 10 * c * rest >> 8;
    const int cost = (n >> 8) * 10 * c + (rest == 0 ? 0 : (walk > share ? walk : share));
    if (counts.n[c - 1] > 0 && cost <= best_cost) { best_cost = cost; best = c; }
  }
  return best;
}

}  // namespace evict
