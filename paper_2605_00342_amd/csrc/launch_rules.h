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

}  // namespace evict
