// Weight-streaming skinny GEMM for gfx950: out[token][row] = sum_k W[row][k] * X[token][k]
// with at most a few dozen tokens per weight matrix, so the kernel is bound by reading W
// from HBM exactly once. Used for the QKV / output projections and for the grouped expert
// GEMMs over the union of activated experts (Sec. 2.2, Eq. 5).
//
// Layout: W is pre-packed into 16-row strips; a strip is nkb consecutive 1 KiB blocks, one
// block = one wavefront-wide 16-byte load = one MFMA operand (64 bytes of each of 16 rows).
// A workgroup of 8 wavefronts owns a contiguous range of strips (contiguous in memory, so
// the stream is sequential); the contraction range of a strip is split across the 8
// wavefronts, each keeping its slice of the token operand in registers for as long as the
// expert does not change. Partial tiles meet in LDS, one wavefront (rotating) sums them and
// runs the epilogue. The whole work list (union experts x strips) is cut into equal
// contiguous ranges on the device, so no host knowledge of the union size is needed.
#pragma once
#include <type_traits>

#include "device_utils.h"

namespace evict {

// SWIGLU and F32 (fp32 rows, the down projection) are grouped by expert, the others dense; ROWS: fp32 rows of a dense matrix (score
// rows). What the operand is must be known at compile time: with one instance for both kinds of fp32 rows and a stride chosen
// when it runs, score rows took up to 14 % longer (128256 rows of 96 blocks, 1 token, us: 150 -> 131; 32-bit storage, 32000 of 64 34.6 -> 30.8).
// ARGMAX_WG, ROWS_WG: the same, kept by the workgroup until its strips are done (likewise: the way that is not taken, left in as a branch, costs
// score rows of 24 blocks 2 to 5 %).
enum { EPI_QKV = 0, EPI_RESID = 1, EPI_SWIGLU = 2, EPI_F32 = 3, EPI_ARGMAX = 4, EPI_ROWS = 5, EPI_ARGMAX_WG = 6, EPI_ROWS_WG = 7 };

// One slot of the device-side work list = one activated expert and one tile of up to 16 of its
// tokens: the expert, where the tile sits in the grouped order, how many tokens it has, how many
// tiles the expert has, and the token ids of the tile's first positions (so that a workgroup
// learns everything it needs to start loading from one 64-byte record).
constexpr int kWorkToks = 12;
struct WorkRec {
  int expert, p0, ntok, pad;
  int tok[kWorkToks];
};

struct GemmArgs {
  const u32x4* W;        // packed weights
  const u32x4* W_shared; // grouped: packed weights of the always-on shared experts (expert ids >= n_routed)
  int n_routed;          // grouped: number of routed experts E
  long long group_stride;  // u32x4 elements between experts
  int n_strips;          // 16-row strips per matrix (gate/up interleaved: 2 per 16 rows of F)
  int nkb;               // 1 KiB blocks per strip
  const void* X;         // token operand, storage dtype; grouped: rows, dense: operand blocks (operand_at)
  long long ldx_bytes;   // grouped: bytes between rows of X
  int x_shift;           // dense: operand_shift of the call's tokens
  int grouped;           // 0: one matrix, tokens 0..T-1; 1: one matrix per union expert
  const int* union_count;  // grouped: [0] number of work slots (expert x token tile), [2] units per chunk for them (gateup_chunk)
  const WorkRec* work;   // per union slot (see WorkRec)
  int chunk_units;       // grouped: units per chunk (divides the units per expert); 0: as union_count[2] says (steps of 128 blocks)
  const int* tok_of_pos; // token of each grouped position (perm[p] / k)
  int x_by_token;        // grouped: 1 -> X row = tok_of_pos[p], 0 -> X row = p
  int T;                 // dense: token rows (upper bound when T_dev is set)
  const int* T_dev;      // dense: nullptr, or device word holding the actual number of token rows (<= T)
  int dense_tiles;       // dense: workgroups per strip, each taking 16*NT tokens
  int dense_units;       // dense: consecutive strips a workgroup takes (its weight loads run ahead across them)
  int prefetch;          // host-side choice of the kernel variant: 3 = no compile-time step counts (measurement knob)
  int wave_strip;        // host-side: grouped fp32-output GEMM may use gemm_wave_strip_kernel
  int nt_loads;          // host-side choice of the kernel variant: 1 = weights fetched with non-temporal loads
  int lds_dma;           // 1: strip-pair gate/up kernel stages its token operand with direct global-to-LDS loads
  int down_ws;           // gemm_wave_strip_kernel: strips (wavefronts) per workgroup, 8 or 16
  int pair_tiles;        // 1: gemm_wave_strip_kernel with two token tiles takes them from two consecutive 16-token records
  int rows_lds;          // ROWS_WG: bytes of LDS for the scores of all strips of a workgroup
  void* out0;            // QKV: q; RESID: h; SWIGLU: act; F32: y; ROWS: scores; ARGMAX: best value per token and strip, or workgroup (best_kept), [T][ldo]
  void* out1;            // QKV: k_new; ARGMAX: row index of the best value
  void* out2;            // QKV: v_new
  long long ldo;         // elements between output rows (RESID / SWIGLU / F32 / ROWS)
  const void* resid;     // RESID: residual rows, same layout as out0
  const float* rope_cs;  // QKV: [T][D] cos | sin
  int Hq, Hkv, D;
};

constexpr int kGemmWaves = 8;
constexpr int kGemmThreads = kGemmWaves * 64;

// Arg max with the candidates kept by the wavefronts until a workgroup's strips are done: always with two token tiles (1 token, us: 9496 strips of
// 32 blocks 69 strip by strip, 107 this way, 2000 of 32 20 against 27; but two tiles, 32 tokens, 9496 strips of 32 blocks 75 -> 57, 48 blocks 126 -> 104),
// with one where lm_keeps_best says so.
template <int EPI, int NT> constexpr bool best_kept() { return EPI == EPI_ARGMAX_WG || (EPI == EPI_ARGMAX && NT == 2); }

// Score rows of a workgroup's strips, kept in LDS until its weights have been streamed. (Stored strip by strip, a wavefront's next weights wait
// behind its stores, as one counter in order of issue covers both: 151936 rows of 64 blocks, 32 tokens, us: 113 -> 99.)
constexpr int kRowsLdsMax = 96 * 1024;
// where quarter q (rows 4q .. 4q + 3) of a strip's row block for token column n lies: columns XORed so that 16 lanes which read
// neighbouring strips' quarters of one token meet 16 different places
__device__ __forceinline__ int rows_lds_at(int strip, int q, int n) { return q * 16 + (n ^ ((strip * 4 + q) & 15)); }

// KBW: 1 KiB blocks a wavefront takes per step (EXACT: every step has exactly KBW, no masking);
// PF: steps of weight loads kept in flight; NT: 16-token tiles held in registers; IS: strips
// taken per step (one partial-tile exchange per IS strips).
// NS > 0: steps per segment known at compile time (the step loop is unrolled, so the rolling refill of
// the weight registers is unconditional and every wait is by exact queue position).
// NTL: weights are fetched with non-temporal loads (read once, or by the neighbouring token tile at about the
// same time: kept out of the caches' way). Ordinary loads stream about 15 % slower here and leave L2 and the
// memory-side cache full of weights nobody reads again, which slows the kernels that follow (measured). This is
// a compile-time choice on purpose: a run-time choice per load between a non-temporal and an ordinary load of
// the same address is folded by the compiler into one ordinary load. (Measured too: ordinary loads for all but
// the last token tile of an expert, so that later tiles find the weights in L2, lose more in the following
// kernels than they save in this one.)
// Registers: two workgroups per CU where one token tile, or short strips, leave it at 128 of them. (Arg max of 24 blocks, two token tiles,
// takes 137 if it may, and two rounds of workgroups then run one behind the other: 48 tokens, 3142 strips 29.1 us,
// 26.6 with candidates stored strip by strip, 22.7 with 128; 6250 strips 42.5, 38.6, 31.9.)
template <typename ST, int NT, int KBW, int PF, int EPI, bool EXACT, int IS = 1, int NS = 0, bool NTL = false>
__global__ __launch_bounds__(kGemmThreads) __attribute__((amdgpu_waves_per_eu((NT == 1 && KBW <= 8) || (EPI == EPI_ARGMAX && KBW <= 3) ? 4 : 2))) void gemm_stream_kernel(const GemmArgs a) {
  constexpr int SPU = (EPI == EPI_SWIGLU) ? 2 : 1;  // strips per unit of work
  static_assert(EPI != EPI_SWIGLU || IS == 1, "gate/up strips are exchanged one at a time");
  __shared__ f32x4 s_part[2][kGemmWaves][IS * NT][64];
  extern __shared__ __attribute__((aligned(16))) f32x4 s_rows[];  // ROWS_WG: a.rows_lds

  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);  // wavefront index, known uniform
  const int upg = a.n_strips / SPU;
  const int nkb = a.nkb;
  constexpr int CB = EXACT && KBW > 8 ? KBW * kGemmWaves : 64;  // contraction blocks per step of the workgroup
  const int nchunks = (nkb + CB - 1) / CB;
  int parity = 0;

  // One segment = `nunits` consecutive units (strips, or gate/up strip pairs) of one weight
  // matrix, applied to the tokens [tok_begin, min(ntok, tok_limit)) of its group.
  auto run_segment = [&](auto nt_tag, int grp, int unit_in_grp, int nunits, int tok_begin, int tok_limit) {
    constexpr bool once = decltype(nt_tag)::value;
    const int strip0 = unit_in_grp * SPU;
    const int nitems = nunits * SPU;
    int p0 = 0, ntok = a.grouped ? 0 : dyn_tokens(a.T_dev, a.T);
    int tok_early = 0;  // token id from the work record (grouped, first kWorkToks positions)
    const u32x4* wbase = a.W;
    if (a.grouped) {
      // one hop: the record (scalar) and this lane's token id (vector) are fetched together
      const WorkRec* rec = a.work + grp;
      const int lc = lane & 15;
      tok_early = rec->tok[lc < kWorkToks ? lc : kWorkToks - 1];  // entries past ntok repeat the last token
      p0 = rec->p0;
      ntok = rec->ntok;
      const int ex = rec->expert;
      wbase = ex < a.n_routed ? a.W + (long long)ex * a.group_stride : a.W_shared + (long long)(ex - a.n_routed) * a.group_stride;
    }
    const int nsteps = NS > 0 ? NS : (nitems / IS) * nchunks;  // nitems is a multiple of IS (host-checked)

    const int tok_end = ntok < tok_limit ? ntok : tok_limit;
    for (int tok0 = tok_begin; tok0 < tok_end; tok0 += 16 * NT) {
      u32x4 A[PF][IS * KBW];
      u32x4 Bf[NT][KBW];
      f32x4 acc[IS][NT];
      f32x4 gate[NT];
      f32x4 pre0[IS * NT], pre1[IS * NT];  // epilogue operands requested ahead (QKV / RESID)
      float best_v[NT];  // ARGMAX
      int best_i[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) { best_v[t] = -INFINITY; best_i[t] = 0x7fffffff; }
#pragma unroll
      for (int q = 0; q < IS * NT; ++q) pre0[q] = pre1[q] = f32x4{0, 0, 0, 0};
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        gate[t] = f32x4{0, 0, 0, 0};
#pragma unroll
        for (int i = 0; i < IS; ++i) acc[i][t] = f32x4{0, 0, 0, 0};
      }

      // block range of this wavefront inside chunk c: [b0, b0 + nb)
      auto range = [&](int c, int& b0, int& nb) {
        if (EXACT) {
          b0 = c * CB + w * KBW;
          nb = KBW;
        } else {
          int cb = nkb - c * 64;
          cb = cb > 64 ? 64 : cb;
          b0 = c * 64 + (w * cb) / kGemmWaves;
          nb = c * 64 + ((w + 1) * cb) / kGemmWaves - b0;
        }
      };
      auto issue = [&](u32x4(&dst)[IS * KBW], int step) {
        const int it = step / nchunks, c = step - it * nchunks;
        int b0, nb;
        range(c, b0, nb);
#pragma unroll
        for (int i = 0; i < IS; ++i) {
          const u32x4* p = wbase + ((long long)(strip0 + it * IS + i) * nkb + b0) * 64 + lane;
#pragma unroll
          for (int j = 0; j < KBW; ++j)
            if (EXACT || j < nb) dst[i * KBW + j] = once ? __builtin_nontemporal_load(p + j * 64) : p[j * 64];
        }
      };
      // weights first: their addresses need nothing but the expert id
#pragma unroll
      for (int r = 0; r < PF; ++r)
        if (r < nsteps) issue(A[r], r);

      // token operand of this lane's column in each tile
      constexpr bool kDense = EPI != EPI_F32 && EPI != EPI_SWIGLU;
      const char* xrow[NT];
      uint32_t xoff[NT];  // dense: offset from a base that is the same for all lanes
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        int col = tok0 + t * 16 + (lane & 15);
        if (col > ntok - 1) col = ntok - 1;  // padded columns repeat the last token; never stored
        long long row = col;
        if (a.grouped) {
          if (!a.x_by_token) row = p0 + col;
          else row = (t == 0 && tok0 == 0 && (lane & 15) < kWorkToks) ? tok_early : a.tok_of_pos[p0 + col];
        }
        if (kDense) xoff[t] = operand_at(col, lane >> 4, nkb, a.x_shift);
        else xrow[t] = (const char*)a.X + row * a.ldx_bytes + (lane >> 4) * 16;
      }
      const int xstep = kDense ? 64 << a.x_shift : 64;  // bytes between a row's blocks
      auto load_b = [&](int c) {
        int b0, nb;
        range(c, b0, nb);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          const char* base = (kDense ? (const char*)a.X : xrow[t]) + (long long)b0 * xstep;
#pragma unroll
          for (int j = 0; j < KBW; ++j)
            if (EXACT || j < nb)
              Bf[t][j] = *reinterpret_cast<const u32x4*>(kDense ? base + j * xstep + xoff[t] : base + j * 64);
        }
      };
      if (nchunks == 1) load_b(0);

#pragma unroll
      for (int s0 = 0; s0 < (NS > 0 ? NS : nsteps); s0 += PF) {
#pragma unroll
        for (int r = 0; r < PF; ++r) {
          const int step = s0 + r;
          if (step < nsteps) {
            const int it = step / nchunks, c = step - it * nchunks;
            if (nchunks > 1) load_b(c);
            if ((EPI == EPI_QKV || EPI == EPI_RESID) && c == 0) {
              // the wavefront that will reduce this strip requests what its epilogue needs (rotation
              // table entries, residual values) now, so that round trip hides behind the weight stream
              const int rb0 = unit_in_grp + it / SPU;
#pragma unroll
              for (int q = 0; q < IS * NT; ++q) {
                if (w == ((rb0 + q) & (kGemmWaves - 1))) {
                  const int t = q % NT;
                  const int strip = strip0 + it * IS + q / NT;
                  const int col = tok0 + t * 16 + (lane & 15);
                  const int tokc = col < ntok ? col : 0;
                  if (EPI == EPI_RESID) {
                    pre0[q] = load4<ST>(a.resid, (long long)tokc * a.ldo + strip * 16 + (lane >> 4) * 4);
                  } else {
                    const int spd = a.D >> 4;
                    const int head = strip / spd, js = strip - head * spd;
                    const int idx = js * 8 + ((lane >> 4) & 1) * 4;
                    const float* cs = a.rope_cs + (long long)tokc * a.D;
                    pre0[q] = *reinterpret_cast<const f32x4*>(cs + idx);
                    pre1[q] = *reinterpret_cast<const f32x4*>(cs + (a.D >> 1) + idx);
                  }
                }
              }
            }
            int b0, nb;
            range(c, b0, nb);
            if (EXACT && PF == 1 && NS > 0) {
              // rolling refill: the block of the next step goes into a register as soon as the MFMA has
              // consumed it, so about KBW loads stay in flight instead of falling to none at the end of
              // a step (same registers; the queue position of every load stays known at compile time)
              const bool more = step + 1 < nsteps;
              const int itn = (step + 1) / nchunks, cn = (step + 1) - itn * nchunks;
              const long long boff = (long long)(cn * CB + w * KBW);
#pragma unroll
              for (int i = 0; i < IS; ++i) {
                const u32x4* pn = wbase + ((long long)(strip0 + itn * IS + i) * nkb + boff) * 64 + lane;
#pragma unroll
                for (int j = 0; j < KBW; ++j) {
#pragma unroll
                  for (int t = 0; t < NT; ++t) acc[i][t] = mfma_block<ST>(A[r][i * KBW + j], Bf[t][j], acc[i][t]);
                  if (more) A[r][i * KBW + j] = once ? __builtin_nontemporal_load(pn + j * 64) : pn[j * 64];
                  __builtin_amdgcn_sched_barrier(0);  // the refill stays right behind its MFMA
                }
              }
            } else {
#pragma unroll
              for (int i = 0; i < IS; ++i)
#pragma unroll
                for (int j = 0; j < KBW; ++j)
                  if (EXACT || j < nb) {
#pragma unroll
                    for (int t = 0; t < NT; ++t) acc[i][t] = mfma_block<ST>(A[r][i * KBW + j], Bf[t][j], acc[i][t]);
                  }
              if (step + PF < nsteps) issue(A[r], step + PF);
            }
            if (c == nchunks - 1) {
              // strip finished: exchange partial tiles, one wavefront reduces and stores
#pragma unroll
              for (int i = 0; i < IS; ++i)
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                  s_part[parity][w][i * NT + t][lane] = acc[i][t];
                  acc[i][t] = f32x4{0, 0, 0, 0};
                }
              lds_barrier();
              // tile q = (strip i of the step, token tile t) is summed by wavefront (rbase + q) % 8
              const int rbase = unit_in_grp + it / SPU;
#pragma unroll
              for (int q = 0; q < IS * NT; ++q) {
                if (w == ((rbase + q) & (kGemmWaves - 1))) {
                  const int t = q % NT;
                  const int strip = strip0 + it * IS + q / NT;
                  f32x4 sum = s_part[parity][0][q][lane];
#pragma unroll
                  for (int ww = 1; ww < kGemmWaves; ++ww) sum += s_part[parity][ww][q][lane];
                  const int col = tok0 + t * 16 + (lane & 15);
                  const bool valid = col < ntok;
                  const int m0 = (lane >> 4) * 4;  // first of this lane's 4 rows in the strip
                  if (best_kept<EPI, NT>()) {
                    // best of this lane's rows in all strips of this wavefront, the lowest row on equal values
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                      const int row = strip * 16 + m0 + i;
                      if (sum[i] > best_v[t] || (sum[i] == best_v[t] && row < best_i[t])) { best_v[t] = sum[i]; best_i[t] = row; }
                    }
                  } else if (EPI == EPI_ARGMAX) {
                    // best of this lane's 4 rows (lowest row on equal values), then across the 4
                    // lanes that hold the other rows of the same token
                    float bv = sum[0];
                    int bi = strip * 16 + m0;
#pragma unroll
                    for (int i = 1; i < 4; ++i)
                      if (sum[i] > bv) { bv = sum[i]; bi = strip * 16 + m0 + i; }
#pragma unroll
                    for (int o = 16; o <= 32; o <<= 1) {
                      const float ov = __shfl_xor(bv, o);
                      const int oi = __shfl_xor(bi, o);
                      if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
                    }
                    if (valid && lane < 16) {
                      ((float*)a.out0)[(long long)col * a.ldo + strip] = bv;
                      ((int*)a.out1)[(long long)col * a.ldo + strip] = bi;
                    }
                  } else if (EPI == EPI_ROWS_WG) {
                    s_rows[((strip - strip0) * NT + t) * 64 + rows_lds_at(strip - strip0, lane >> 4, lane & 15)] = sum;
                  } else if (EPI == EPI_F32 || EPI == EPI_ROWS) {
                    if (valid) {
                      const long long orow = a.grouped ? (p0 + col) : col;
                      *reinterpret_cast<f32x4*>((float*)a.out0 + orow * a.ldo + strip * 16 + m0) = sum;
                    }
                  } else if (EPI == EPI_RESID) {
                    if (valid) {
                      const long long o = (long long)col * a.ldo + strip * 16 + m0;
                      store4<ST>(a.out0, o, pre0[q] + sum);
                    }
                  } else if (EPI == EPI_SWIGLU) {
                    if ((it & 1) == 0) {
                      gate[t] = sum;  // gate strip; its up strip is the next item
                    } else if (valid) {
                      f32x4 g = gate[t], r4;
#pragma unroll
                      for (int i = 0; i < 4; ++i) r4[i] = (g[i] / (1.0f + __expf(-g[i]))) * sum[i];
                      const long long orow = a.grouped ? (p0 + col) : col;
                      store4<ST>(a.out0, orow * a.ldo + (strip >> 1) * 16 + m0, r4);
                    }
                  } else {  // EPI_QKV: rotate pairs (i, i + D/2), which sit 32 lanes apart
                    const int spd = a.D >> 4;  // strips per head
                    const int head = strip / spd, js = strip - head * spd;
                    const int half = a.D >> 1;
                    const int g4 = lane >> 4;
                    const int idx = js * 8 + (g4 & 1) * 4;  // index inside the half
                    f32x4 other, r4;
#pragma unroll
                    for (int i = 0; i < 4; ++i) other[i] = __shfl_xor(sum[i], 32);
                    const bool rot = head < a.Hq + a.Hkv;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                      const float cv = rot ? pre0[q][i] : 1.0f;
                      const float sv = rot ? pre1[q][i] : 0.0f;
                      r4[i] = (g4 < 2) ? (sum[i] * cv - other[i] * sv) : (sum[i] * cv + other[i] * sv);
                    }
                    if (valid) {
                      const int hrow = (g4 < 2 ? 0 : half) + idx;
                      if (head < a.Hq) {
                        store4<ST>(a.out0, ((long long)col * a.Hq + head) * a.D + hrow, r4);
                      } else if (head < a.Hq + a.Hkv) {
                        store4<ST>(a.out1, ((long long)col * a.Hkv + (head - a.Hq)) * a.D + hrow, r4);
                      } else {
                        store4<ST>(a.out2, ((long long)col * a.Hkv + (head - a.Hq - a.Hkv)) * a.D + hrow, r4);
                      }
                    }
                  }
                }
              }
              parity ^= 1;
            }
          }
        }
      }
      if (EPI == EPI_ROWS_WG) {
        lds_barrier();
        const int live = tok_end - tok0 < 16 * NT ? tok_end - tok0 : 16 * NT, per_tok = nitems * 4;
        for (int i = tid; i < live * per_tok; i += kGemmThreads) {
          const int n = i / per_tok, r = i - n * per_tok, strip = r >> 2, q = r & 3;
          const f32x4 v = s_rows[(strip * NT + (n >> 4)) * 64 + rows_lds_at(strip, q, n & 15)];
          *reinterpret_cast<f32x4*>((float*)a.out0 + (long long)(tok0 + n) * a.ldo + strip0 * 16 + r * 4) = v;
        }
      }
      if (best_kept<EPI, NT>()) {
        // one candidate per token and workgroup: the wavefronts' bests, then those of the 4 lanes that hold other rows of a token.
        // (151936 rows of 64 blocks, 32 tokens, us: with an exchange between lanes and a store at every strip 102, 6.1 TB/s, and 6.4
        // for the best of 9496 candidates; this way 91, 6.8 TB/s, and 4.8 for the best of 256)
#pragma unroll
        for (int t = 0; t < NT; ++t) s_part[parity][w][t][lane] = f32x4{best_v[t], __int_as_float(best_i[t]), 0.0f, 0.0f};
        lds_barrier();
        if (w < NT) {
          float bv = -INFINITY;
          int bi = 0x7fffffff;
          auto take = [&](float ov, int oi) {
            if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
          };
#pragma unroll
          for (int ww = 0; ww < kGemmWaves; ++ww) {
            const f32x4 o = s_part[parity][ww][w][lane];
            take(o[0], __float_as_int(o[1]));
          }
#pragma unroll
          for (int o = 16; o <= 32; o <<= 1) take(__shfl_xor(bv, o), __shfl_xor(bi, o));
          const int col = tok0 + w * 16 + lane;
          if (lane < 16 && col < ntok) {
            const long long at = (long long)col * a.ldo + unit_in_grp / a.dense_units;
            ((float*)a.out0)[at] = bv;
            ((int*)a.out1)[at] = bi;
          }
        }
        parity ^= 1;
      }
    }
  };

  if (a.grouped) {
    // Device-side work list: union experts x units, cut into chunks of `chunk_units` units that
    // never straddle an expert. Chunks are dealt round-robin to the workgroups; all chunks cost
    // the same, so this stays balanced for any union size without the host knowing it.
    const int slots = *a.union_count;
    const int cu = CB > 64 && a.chunk_units == 0 ? a.union_count[2] : a.chunk_units;
    const int cpg = upg / cu;
    const int total = slots * cpg;
    for (int chunk = blockIdx.x; chunk < total; chunk += gridDim.x) {
      // (the token tiles of one expert are consecutive slots: with cpg a multiple of 8 their
      // chunks land on the same XCD, whose L2 serves the second reader of the weights)
      const int slot = chunk / cpg, uc = chunk - slot * cpg;
      run_segment(std::integral_constant<bool, NTL>{}, slot, uc * cu, cu, 0, 0x7fffffff);
    }
  } else {
    // one workgroup per (strip, token tile). Workgroup ids go round-robin over the 8 XCDs, so
    // the tiles of one strip are given ids 8 apart: they share an L2 and read the strip from
    // HBM once.
    const unsigned xcd = blockIdx.x & 7u, i = blockIdx.x >> 3;
    const unsigned tile = i % (unsigned)a.dense_tiles;
    const unsigned du = a.dense_units > 0 ? (unsigned)a.dense_units : 1u;
    const unsigned unit = ((i / (unsigned)a.dense_tiles) * 8u + xcd) * du;
    if (unit >= (unsigned)upg) return;
    const unsigned nu = unit + du <= (unsigned)upg ? du : (unsigned)upg - unit;
    run_segment(std::integral_constant<bool, NTL>{}, 0, (int)unit, (int)nu, (int)tile * 16 * NT, (int)(tile + 1) * 16 * NT);
  }
}

// ------------------------------------------------------------------------------------
// Second decomposition for grouped GEMMs with many strips and a short contraction (the down
// projections: d/16 strips of F columns per expert): one strip per wavefront over the whole
// contraction range, so no partial tiles are exchanged and nothing synchronises the wavefronts
// after the token operand has been staged. The 16 x K token operand of the slot sits in LDS as
// ready-made MFMA operand blocks; weight blocks travel through a rolling window of WIN
// registers per lane (WIN KiB in flight per wavefront); NB operand blocks are staged per wavefront and
// pass. A workgroup takes WS consecutive strips
// of one slot (chunk); chunks are dealt round-robin like in gemm_stream_kernel.
// Output: fp32 rows y[p0 + column][strip * 16 + ...] (the EPI_F32 contract). NTW token tiles of 16
// per slot (the work list is built with tiles of 16 * NTW tokens).
// LDS: NTW * nkb KiB (dynamic).
// ------------------------------------------------------------------------------------
// NKB > 0 fixes the number of contraction blocks at compile time: every loop between the issue of
// a weight load and its use is then fully unrolled, which is what lets the compiler wait for a
// load by its exact position in the in-order queue (with run-time trip counts it has to drain the
// queue before the first MFMA, and the window stops rolling).
template <typename ST, int WIN, int NB, bool EXACT, int NTW = 1, int WS = 8, int NKB = 0, bool NTL = false>
__global__ __launch_bounds__(WS * 64) __attribute__((amdgpu_waves_per_eu(4))) void gemm_wave_strip_kernel(const GemmArgs a) {
  extern __shared__ __attribute__((aligned(16))) u32x4 s_b[];  // [NTW token tiles][nkb][64]
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nkb = NKB > 0 ? NKB : a.nkb;
  const int cpg = a.n_strips / WS;  // chunks per slot (host-checked: divides)
  const int total = *a.union_count * cpg;
  bool first = true;
  // one chunk; nt_tag: non-temporal weight loads (see gemm_stream_kernel)
  auto run_chunk = [&](auto nt_tag, int chunk) {
    constexpr bool once = decltype(nt_tag)::value;
    const int slot = chunk / cpg, strip = (chunk - slot * cpg) * WS + w;
    const WorkRec* rec = a.work + slot;
    const int p0 = rec->p0, ex = rec->expert;
    int ntok = rec->ntok;
    if (NTW == 2 && a.pair_tiles) {
      // The work list holds 16-token tiles; the tiles of an expert are consecutive records over consecutive
      // positions. An even tile takes its successor along (one weight stream for both), an odd one is done.
      const int ntile = rec->pad & 0xFFFF, ti = rec->pad >> 16;
      if (ti & 1) return;
      if (ti + 1 < ntile) ntok += rec[1].ntok;
    }
    const u32x4* wbase = ex < a.n_routed ? a.W + (long long)ex * a.group_stride
                                         : a.W_shared + (long long)(ex - a.n_routed) * a.group_stride;
    // token operand first, weights behind it: the in-order load counter then lets the operand
    // be consumed while the weight window is still in flight
    const char* xrow[NTW];
    bool valid[NTW];
#pragma unroll
    for (int t = 0; t < NTW; ++t) {
      int col = t * 16 + (lane & 15);
      valid[t] = col < ntok;
      col = valid[t] ? col : ntok - 1;  // padded columns repeat the last token; never stored
      const long long xr = a.x_by_token ? a.tok_of_pos[p0 + col] : p0 + col;
      xrow[t] = (const char*)a.X + xr * a.ldx_bytes + (lane >> 4) * 16;
    }
    constexpr int BMAX = NB;  // operand blocks a wavefront stages per pass and token tile
    const u32x4* wp = wbase + (long long)strip * nkb * 64 + lane;
    u32x4 A[WIN];
#pragma unroll
    for (int kb0 = 0; kb0 < (NKB > 0 ? NKB : nkb); kb0 += BMAX * WS) {
      u32x4 bst[NTW][BMAX];
#pragma unroll
      for (int t = 0; t < NTW; ++t)
#pragma unroll
        for (int i = 0; i < BMAX; ++i) {
          const int kb = kb0 + i * WS + w;
          if (kb < nkb && t * 16 < ntok) bst[t][i] = *reinterpret_cast<const u32x4*>(xrow[t] + (long long)kb * 64);
        }
      if (kb0 == 0) {
#pragma unroll
        for (int j = 0; j < WIN; ++j)
          if (EXACT || j < nkb) A[j] = once ? __builtin_nontemporal_load(wp + j * 64) : wp[j * 64];
        if (!first) lds_barrier();  // every wavefront is done with the previous chunk's operand
      }
#pragma unroll
      for (int t = 0; t < NTW; ++t)
#pragma unroll
        for (int i = 0; i < BMAX; ++i) {
          const int kb = kb0 + i * WS + w;
          if (kb < nkb && t * 16 < ntok) s_b[((size_t)t * nkb + kb) * 64 + lane] = bst[t][i];
        }
    }
    lds_barrier();
    first = false;
    f32x4 acc[NTW];
#pragma unroll
    for (int t = 0; t < NTW; ++t) acc[t] = f32x4{0, 0, 0, 0};
#pragma unroll
    for (int j0 = 0; j0 < (NKB > 0 ? NKB : nkb); j0 += WIN) {
#pragma unroll
      for (int jj = 0; jj < WIN; ++jj) {
        const int j = j0 + jj;
        if (EXACT || j < nkb) {
#pragma unroll
          for (int t = 0; t < NTW; ++t)
            if (t == 0 || ntok > 16) acc[t] = mfma_block<ST>(A[jj], s_b[((size_t)t * nkb + j) * 64 + lane], acc[t]);
          if (j + WIN < nkb) A[jj] = once ? __builtin_nontemporal_load(wp + (j + WIN) * 64) : wp[(j + WIN) * 64];
          if (NKB > 0) __builtin_amdgcn_sched_barrier(0);  // keep the refill right behind its MFMA: the window stays full
        }
      }
    }
#pragma unroll
    for (int t = 0; t < NTW; ++t)
      if (valid[t])
        *reinterpret_cast<f32x4*>((float*)a.out0 + (p0 + t * 16 + (lane & 15)) * a.ldo + strip * 16 + (lane >> 4) * 4) = acc[t];
  };
  for (int chunk = blockIdx.x; chunk < total; chunk += gridDim.x) run_chunk(std::integral_constant<bool, NTL>{}, chunk);
}

// ------------------------------------------------------------------------------------
// The same decomposition for the gate/up projections: one (gate strip, up strip) pair per
// wavefront over the whole contraction range (2 x nkb KiB of weights per wavefront and unit),
// the 16 x d token operand of the slot in LDS, two rolling windows of WIN weight blocks (one per
// strip; a token operand block read from LDS feeds both MFMAs), SiLU(g) * u applied in the
// wavefront that owns the pair. WS wavefronts per workgroup share the staged operand; a
// workgroup lives for WS * 2 * nkb KiB of weights, so the stream has no exchange points.
// Requires nkb % WIN == 0, (n_strips / 2) % WS == 0, NTW * nkb KiB of LDS (NTW tiles of 16 tokens per
// work-list slot). Refills go out in runs of 8
// consecutive blocks per strip once the window is 16 deep.
// ------------------------------------------------------------------------------------
template <typename ST, int WIN, int NB, int WS, int NKB = 0, int NTW = 1, bool DMA = false, bool NTL = false>
__global__ __launch_bounds__(WS * 64) __attribute__((amdgpu_waves_per_eu(2))) void gemm_wave_gateup_kernel(const GemmArgs a) {
  static_assert(!DMA || (NTW == 1 && 2 * WIN <= 48), "direct-to-LDS staging: one token tile, window loads countable in vmcnt");
  extern __shared__ __attribute__((aligned(16))) u32x4 s_b[];  // [NTW token tiles][nkb][64]
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nkb = NKB > 0 ? NKB : a.nkb;
  const int cpg = (a.n_strips >> 1) / WS;  // chunks per slot
  const int total = *a.union_count * cpg;
  bool first = true;
  // one chunk; nt_tag: non-temporal weight loads (see gemm_stream_kernel)
  auto run_chunk = [&](auto nt_tag, int chunk) {
    constexpr bool once = decltype(nt_tag)::value;
    const int slot = chunk / cpg, unit = (chunk - slot * cpg) * WS + w;
    const WorkRec* rec = a.work + slot;
    const int lc = lane & 15;
    const int tok_early = rec->tok[lc < kWorkToks ? lc : kWorkToks - 1];
    const int p0 = rec->p0, ntok = rec->ntok, ex = rec->expert;
    const u32x4* wbase = ex < a.n_routed ? a.W + (long long)ex * a.group_stride
                                         : a.W_shared + (long long)(ex - a.n_routed) * a.group_stride;
    // (NTW token tiles of 16 per slot: the work list was built with tiles of 16 * NTW tokens)
    bool valid[NTW];
    const char* xrow[NTW];
#pragma unroll
    for (int t = 0; t < NTW; ++t) {
      int col = t * 16 + lc;
      valid[t] = col < ntok;
      col = valid[t] ? col : ntok - 1;  // padded columns repeat the last token; never stored
      long long xr = p0 + col;
      if (a.x_by_token) xr = (t == 0 && col < kWorkToks) ? tok_early : a.tok_of_pos[p0 + col];
      xrow[t] = (const char*)a.X + xr * a.ldx_bytes + (lane >> 4) * 16;
    }
    // token operand blocks of the first tile first, weights behind them (the in-order load counter lets
    // the operand be consumed while the weight windows are still in flight); a second tile reuses the
    // staging registers once the first is in LDS. DMA: the operand blocks go from global memory straight
    // into LDS (16 bytes per lane, a block = 1 KiB contiguous = exactly the LDS layout), no staging registers.
    u32x4 bst[DMA ? 1 : NB];
    if (DMA) {
      if (!first) lds_barrier();  // every wavefront is done with the previous chunk's operand
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        const int kb = i * WS + w;
        if (kb < nkb)
          __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1)))*)(xrow[0] + (long long)kb * 64),
                                           (void __attribute__((address_space(3)))*)(s_b + (size_t)kb * 64), 16, 0, 0);
      }
    }
    if constexpr (!DMA) {
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        const int kb = i * WS + w;
        if (kb < nkb) bst[i] = *reinterpret_cast<const u32x4*>(xrow[0] + (long long)kb * 64);
      }
    }
    const u32x4* wg = wbase + (long long)(2 * unit) * nkb * 64 + lane;
    const u32x4* wu = wg + (long long)nkb * 64;
    u32x4 Ag[WIN], Au[WIN];
#pragma unroll
    for (int j = 0; j < WIN; ++j) {
      Ag[j] = once ? __builtin_nontemporal_load(wg + j * 64) : wg[j * 64];
      Au[j] = once ? __builtin_nontemporal_load(wu + j * 64) : wu[j * 64];
    }
    if (DMA) {
      // the operand blocks were requested before the 2 * WIN window loads: wait until only those are outstanding
      constexpr int kVm = 2 * WIN;
      __builtin_amdgcn_s_waitcnt((kVm & 0xF) | ((kVm >> 4) << 14) | (0x7 << 4) | (0xF << 8));
    } else if (!first) {
      lds_barrier();  // every wavefront is done with the previous chunk's operand
    }
    if constexpr (!DMA) {
#pragma unroll
      for (int t = 0; t < NTW; ++t) {
        if (t > 0) {
#pragma unroll
          for (int i = 0; i < NB; ++i) {
            const int kb = i * WS + w;
            if (kb < nkb) bst[i] = *reinterpret_cast<const u32x4*>(xrow[t] + (long long)kb * 64);
          }
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) {
          const int kb = i * WS + w;
          if (kb < nkb) s_b[((size_t)t * nkb + kb) * 64 + lane] = bst[i];
        }
      }
    }
    lds_barrier();
    first = false;
    f32x4 accg[NTW], accu[NTW];
#pragma unroll
    for (int t = 0; t < NTW; ++t) accg[t] = accu[t] = f32x4{0, 0, 0, 0};
    constexpr int BURST = WIN >= 16 ? 8 : WIN;  // consecutive blocks requested together (DRAM likes runs)
#pragma unroll
    for (int j0 = 0; j0 < (NKB > 0 ? NKB : nkb); j0 += WIN) {
#pragma unroll
      for (int jj = 0; jj < WIN; ++jj) {
        const int j = j0 + jj;
#pragma unroll
        for (int t = 0; t < NTW; ++t) {
          const u32x4 bf = s_b[((size_t)t * nkb + j) * 64 + lane];
          accg[t] = mfma_block<ST>(Ag[jj], bf, accg[t]);
          accu[t] = mfma_block<ST>(Au[jj], bf, accu[t]);
        }
        if ((jj % BURST) == BURST - 1) {
          // the BURST window entries just consumed are refilled with the blocks WIN further on
          const int r0 = jj - (BURST - 1);
          if (j0 + r0 + WIN < nkb) {
#pragma unroll
            for (int r = 0; r < BURST; ++r)
              Ag[r0 + r] = once ? __builtin_nontemporal_load(wg + (j0 + r0 + r + WIN) * 64) : wg[(j0 + r0 + r + WIN) * 64];
#pragma unroll
            for (int r = 0; r < BURST; ++r)
              Au[r0 + r] = once ? __builtin_nontemporal_load(wu + (j0 + r0 + r + WIN) * 64) : wu[(j0 + r0 + r + WIN) * 64];
          }
          if (NKB > 0) __builtin_amdgcn_sched_barrier(0);  // keep the refills where they are: the windows stay full
        }
      }
    }
#pragma unroll
    for (int t = 0; t < NTW; ++t)
      if (valid[t]) {
        f32x4 r4;
#pragma unroll
        for (int i = 0; i < 4; ++i) r4[i] = (accg[t][i] / (1.0f + __expf(-accg[t][i]))) * accu[t][i];
        store4<ST>(a.out0, (long long)(p0 + t * 16 + lc) * a.ldo + unit * 16 + (lane >> 4) * 4, r4);
      }
  };
  for (int chunk = blockIdx.x; chunk < total; chunk += gridDim.x) run_chunk(std::integral_constant<bool, NTL>{}, chunk);
}

// ------------------------------------------------------------------------------------
// Dense projections with many tokens (QKV, output projection once the call has more than a few
// token tiles): the strip-per-wavefront decomposition of gemm_wave_strip_kernel applied to one
// weight matrix and all T tokens. A workgroup takes WS = 8 consecutive strips (one per wavefront,
// whole contraction range, rolling window of WIN weight blocks per lane) and NTW tiles of 16
// tokens, whose operand blocks it stages in LDS once ([NTW][nkb][64], NTW * nkb KiB); nothing
// is exchanged between wavefronts after that, and every wavefront finishes its 16 x 16 tiles
// itself (QKV: rotation of the pairs (i, i + D/2), which sit 32 lanes apart; output projection:
// residual add). 1-D grid: workgroup ids go round-robin over the 8 XCDs, so the token groups of
// one strip group are given ids 8 apart: they share an L2 and read the strips from HBM once.
// Requires nkb % WIN == 0.
// ------------------------------------------------------------------------------------
template <typename ST, int EPI, int NTW, int WS, int NKB = 0>
__global__ __launch_bounds__(WS * 64) void gemm_dense_strip_kernel(const GemmArgs a) {
  static_assert(EPI == EPI_QKV || EPI == EPI_RESID, "dense projections only");
  constexpr int WIN = 16;
  extern __shared__ __attribute__((aligned(16))) u32x4 s_b[];  // [NTW token tiles][nkb][64]
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nkb = NKB > 0 ? NKB : a.nkb;
  const int T = dyn_tokens(a.T_dev, a.T);
  const unsigned ntg = (unsigned)a.dense_tiles;  // token groups of NTW * 16 tokens
  const unsigned xcd = blockIdx.x & 7u, i = blockIdx.x >> 3;
  const unsigned tg = i % ntg;
  const unsigned sg = (i / ntg) * 8u + xcd;  // strip group
  if (sg * WS >= (unsigned)a.n_strips) return;  // (whole workgroup: no barrier is left waiting)
  const int strip_raw = (int)sg * WS + w;
  const bool active = strip_raw < a.n_strips;  // the last group may be short: its idle wavefronts still stage and wait
  const int strip = active ? strip_raw : a.n_strips - 1;
  const int tok0 = (int)tg * NTW * 16;
  if (tok0 >= T) return;  // (a token group past the call's actual token count: whole workgroup, before any barrier)
  const int lc = lane & 15;

  // token operand first, weights behind it
  const char* xrow[NTW];
  bool valid[NTW];
#pragma unroll
  for (int t = 0; t < NTW; ++t) {
    int col = tok0 + t * 16 + lc;
    valid[t] = active && col < T;
    col = col < T ? col : T - 1;  // padded columns repeat the last token; never stored
    xrow[t] = (const char*)a.X + operand_at(col, lane >> 4, nkb, a.x_shift);
  }
  constexpr int BMAX = 4;  // operand blocks a wavefront stages per pass and token tile
  const u32x4* wp = a.W + (long long)strip * nkb * 64 + lane;
  u32x4 A[WIN];
#pragma unroll
  for (int kb0 = 0; kb0 < (NKB > 0 ? NKB : nkb); kb0 += BMAX * WS) {
    u32x4 bst[NTW][BMAX];
#pragma unroll
    for (int t = 0; t < NTW; ++t)
#pragma unroll
      for (int q = 0; q < BMAX; ++q) {
        const int kb = kb0 + q * WS + w;
        if (kb < nkb) bst[t][q] = *reinterpret_cast<const u32x4*>(xrow[t] + ((long long)kb * 64 << a.x_shift));
      }
    if (kb0 == 0) {
#pragma unroll
      for (int j = 0; j < WIN; ++j) A[j] = wp[j * 64];
    }
#pragma unroll
    for (int t = 0; t < NTW; ++t)
#pragma unroll
      for (int q = 0; q < BMAX; ++q) {
        const int kb = kb0 + q * WS + w;
        if (kb < nkb) s_b[((size_t)t * nkb + kb) * 64 + lane] = bst[t][q];
      }
  }
  // what the epilogue needs is requested now, so that its round trip hides behind the weight stream
  f32x4 pre0[NTW], pre1[NTW];
#pragma unroll
  for (int t = 0; t < NTW; ++t) {
    const int col = tok0 + t * 16 + lc;
    const int tokc = col < T ? col : 0;
    if (EPI == EPI_RESID) {
      pre0[t] = load4<ST>(a.resid, (long long)tokc * a.ldo + strip * 16 + (lane >> 4) * 4);
      pre1[t] = f32x4{0, 0, 0, 0};
    } else {
      const int spd = a.D >> 4;
      const int head = strip / spd, js = strip - head * spd;
      const int idx = js * 8 + ((lane >> 4) & 1) * 4;
      const float* cs = a.rope_cs + (long long)tokc * a.D;
      pre0[t] = *reinterpret_cast<const f32x4*>(cs + idx);
      pre1[t] = *reinterpret_cast<const f32x4*>(cs + (a.D >> 1) + idx);
    }
  }
  lds_barrier();
  f32x4 acc[NTW];
#pragma unroll
  for (int t = 0; t < NTW; ++t) acc[t] = f32x4{0, 0, 0, 0};
  // operand blocks are requested from LDS PD steps ahead of their MFMAs (ring of registers), so the LDS
  // latency hides behind the matrix work of the steps in between
  constexpr int PD = 4;
  static_assert(WIN % PD == 0, "ring positions must repeat with the window");
  u32x4 bq[PD][NTW];
#pragma unroll
  for (int p = 0; p < PD; ++p)
#pragma unroll
    for (int t = 0; t < NTW; ++t) bq[p][t] = s_b[((size_t)t * nkb + p) * 64 + lane];
#pragma unroll
  for (int j0 = 0; j0 < (NKB > 0 ? NKB : nkb); j0 += WIN) {
#pragma unroll
    for (int jj = 0; jj < WIN; ++jj) {
      const int j = j0 + jj;
#pragma unroll
      for (int t = 0; t < NTW; ++t) acc[t] = mfma_block<ST>(A[jj], bq[jj % PD][t], acc[t]);
      if (j + PD < nkb) {
#pragma unroll
        for (int t = 0; t < NTW; ++t) bq[jj % PD][t] = s_b[((size_t)t * nkb + j + PD) * 64 + lane];
      }
      if (j + WIN < nkb) A[jj] = wp[(j + WIN) * 64];
      if (NKB > 0) __builtin_amdgcn_sched_barrier(0);  // keep the refills right behind their MFMA: window and ring stay full
    }
  }
  const int m0 = (lane >> 4) * 4;  // first of this lane's 4 rows in the strip
#pragma unroll
  for (int t = 0; t < NTW; ++t) {
    const int col = tok0 + t * 16 + lc;
    const f32x4 sum = acc[t];
    if (EPI == EPI_RESID) {
      if (valid[t]) store4<ST>(a.out0, (long long)col * a.ldo + strip * 16 + m0, pre0[t] + sum);
    } else {  // rotate pairs (i, i + D/2), which sit 32 lanes apart
      const int spd = a.D >> 4;  // strips per head
      const int head = strip / spd, js = strip - head * spd;
      const int half = a.D >> 1;
      const int g4 = lane >> 4;
      const int idx = js * 8 + (g4 & 1) * 4;  // index inside the half
      f32x4 other, r4;
#pragma unroll
      for (int q = 0; q < 4; ++q) other[q] = __shfl_xor(sum[q], 32);
      const bool rot = head < a.Hq + a.Hkv;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float cv = rot ? pre0[t][q] : 1.0f;
        const float sv = rot ? pre1[t][q] : 0.0f;
        r4[q] = (g4 < 2) ? (sum[q] * cv - other[q] * sv) : (sum[q] * cv + other[q] * sv);
      }
      if (valid[t]) {
        const int hrow = (g4 < 2 ? 0 : half) + idx;
        if (head < a.Hq) {
          store4<ST>(a.out0, ((long long)col * a.Hq + head) * a.D + hrow, r4);
        } else if (head < a.Hq + a.Hkv) {
          store4<ST>(a.out1, ((long long)col * a.Hkv + (head - a.Hq)) * a.D + hrow, r4);
        } else {
          store4<ST>(a.out2, ((long long)col * a.Hkv + (head - a.Hq - a.Hkv)) * a.D + hrow, r4);
        }
      }
    }
  }
}

// ------------------------------------------------------------------------------------
// Tiled GEMM for many tokens per weight matrix: WS wavefronts take WS * NS consecutive strips (NS per wavefront, NS = 2
// for a gate / up pair) and up to 16 * NT tokens at once. The weight blocks of a strip go from global memory straight
// into the registers of the one wavefront that owns the strip (packed layout: a block is one coalesced load and one
// MFMA operand), a rolling window of WIN blocks per strip; the token operand, which all wavefronts share, goes through
// LDS in stages of WS contraction blocks, two buffers, each wavefront fetching one block of every token tile D stages
// ahead (loads return in order: an operand stage is behind the weights requested before it, so with short stages one
// stage ahead exposes the latency of memory in each). So LDS holds 2 * NT * WS KiB whatever the contraction length, an
// expert's weights are fetched once for all of its (up to 16 * NT) tokens, and every LDS fragment feeds NS MFMAs, every
// weight register one per token tile.
// Sums: chains of CH contraction blocks, added up in ascending order. Where this kernel stands in for a strip kernel (the
// expert projections of up to 64 blocks) CH is the whole contraction, one chain, and the results are the strip kernel's bit
// for bit. Where it stands in for the contraction split (the layer's projections, the LM head, gate / up of 128 blocks) CH is
// NKB / 8: that kernel adds up eight chains, and one chain eight times as long loses nearly three times as much to rounding
// (score rows against 64-bit sums of the same bf16 operands, relative: 2048 columns 1.02e-7 with eight chains, 2.70e-7 with
// one; 4096 columns 1.37e-7, 3.96e-7); up to 64 blocks these are the same eight chains and the same results bit for bit. The total of the chains so far takes NS * NT more
// fragments: with six token tiles there is room for it only with one set of operand fragments, each refilled behind its last
// MFMA, in place of two (CH < NKB and NT > 4).
// All loops are unrolled over the compile-time block count NKB so that every wait is by queue position.
// Bound by memory up to a few tokens tiles per expert, by the L2 -> CU path beyond. Gate / up of 128 experts 2048 x 768,
// 912 tokens (57 per expert): one 16-token tile at a time re-reads every expert four times, 312 us; this kernel 154 us
// (5.2 TB/s of weights read once); 226 tokens over 111 experts 125 -> 109 us (6.4 TB/s). Down: 145 -> 91, 68 -> 61.5 us.
// ------------------------------------------------------------------------------------
template <int EPI, int NT, int NS, int WS, int WIN, int D, int NKB, bool GROUPED, bool NTL>
__global__ __launch_bounds__(WS * 64) __attribute__((amdgpu_waves_per_eu(2))) void gemm_tile_kernel(const GemmArgs a) {
  static_assert(EPI != EPI_SWIGLU || NS == 2, "a gate / up pair per wavefront");
  constexpr int CH = !GROUPED || NKB > 64 ? NKB / 8 : NKB;  // contraction blocks per chain of sums
  static_assert(NKB % CH == 0, "whole chains");
  constexpr int KC = WS;                        // contraction blocks per stage
  constexpr int NST = (NKB + KC - 1) / KC;      // stages
  constexpr int kShift = 4;                     // dense: blocks of 16 tokens (dense_tiled and lm_tiled ask for more than 8)
  static_assert(WIN <= NKB, "the window holds blocks of one strip");
  extern __shared__ __attribute__((aligned(16))) u32x4 s_x[];  // [2][NT][KC][64]
  const int tid = threadIdx.x, lane = tid & 63, lc = lane & 15;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nsg = (a.n_strips + WS * NS - 1) / (WS * NS);  // strip groups
  bool first = true;
  // Grouped: the rows of an expert's tokens lie anywhere, so a wavefront fetches whole cache lines, 128 bytes (two blocks) of 8
  // rows, and a pair of wavefronts two blocks of 16 rows, instead of half a line of each of 16. In a block in LDS the token is
  // XORed with the 16-byte piece of the line it belongs to, so that the 8 lanes of a line write to 8 bank groups; the readers
  // undo it.
  constexpr bool kLines = GROUPED && NKB <= 64;  // (128 blocks: no registers left for it)
  static_assert(!kLines || (WS % 2 == 0 && NKB % 2 == 0), "whole lines");
  const int wb = kLines ? w & ~1 : w;                            // first block of a stage that this wavefront fetches
  const int lrow = (lane >> 3) + 8 * (w & 1), piece = lane & 7;   // grouped: token of the tile, piece of its line
  const int lput = kLines ? (piece >> 2) * 64 + (piece & 3) * 16 + (lrow ^ piece) : lane;
  const int even = lane ^ (lane >> 4), odd = lane ^ ((lane >> 4) | 4);
  // where a lane reads in a block; without kLines its own place, which the base holds (an offset of its own there costs two registers)
  auto lget = [&](int block) __attribute__((always_inline)) { return kLines ? (block & 1 ? odd : even) : 0; };

  // NTL_: live token tiles of this piece of work
  auto run = [&](auto ntl_tag, const u32x4* wbase, int sg, int p0, int ntok, int tok0) __attribute__((always_inline)) {
    constexpr int NTT = decltype(ntl_tag)::value;
    const int strip_raw = (sg * WS + w) * NS;
    const bool active = strip_raw < a.n_strips;  // the last group may be short: its idle wavefronts still stage and wait
    const int strip = active ? strip_raw : a.n_strips - NS;
    uint32_t xrow[NTT];  // byte offset of the token's row (at most 8192 + shared rows of 8 KiB), or of its part of the first operand block
    bool valid[NTT];
#pragma unroll
    for (int t = 0; t < NTT; ++t) {
      valid[t] = active && tok0 + t * 16 + lc < ntok;
      int col = tok0 + t * 16 + (kLines ? lrow : lc);
      col = col < ntok ? col : ntok - 1;  // padded columns repeat the last token; never stored
      const long long xr = GROUPED ? (a.x_by_token ? a.tok_of_pos[p0 + col] : p0 + col) : col;
      xrow[t] = GROUPED ? (uint32_t)(xr * a.ldx_bytes) + (kLines ? lane & 7 : lane >> 4) * 16 : operand_at(col, lane >> 4, NKB, kShift);
    }
    const u32x4* wp = wbase + (long long)strip * NKB * 64 + lane;
    auto load_w = [&](int i, int j) __attribute__((always_inline)) {
      const u32x4* p = wp + ((long long)i * NKB + j) * 64;
      return NTL ? __builtin_nontemporal_load(p) : *p;
    };
    u32x4 st[D][NTT], A[NS][WIN];
    auto fetch = [&](int s) __attribute__((always_inline)) {
      if (s * KC + KC <= NKB || s * KC + wb < NKB) {
#pragma unroll
        for (int t = 0; t < NTT; ++t) st[s % D][t] = *reinterpret_cast<const u32x4*>((const char*)a.X + (s * KC + wb) * (GROUPED ? 64 : 64 << kShift) + xrow[t]);
      }
    };
    auto put = [&](int s) __attribute__((always_inline)) {
      if (s * KC + KC <= NKB || s * KC + wb < NKB) {
#pragma unroll
        for (int t = 0; t < NTT; ++t) s_x[(((s & 1) * NT + t) * KC + wb) * 64 + lput] = st[s % D][t];
      }
    };
    // token operand first, weights behind it: the in-order load counter lets the operand be consumed while the weights fly
    fetch(0);
#pragma unroll
    for (int j = 0; j < WIN; ++j)
#pragma unroll
      for (int i = 0; i < NS; ++i) A[i][j] = load_w(i, j);
#pragma unroll
    for (int s = 1; s < D; ++s)
      if (s < NST) fetch(s);
    if (!first) lds_barrier();  // every wavefront is done with the previous piece's operand
    first = false;
    put(0);
    lds_barrier();
    f32x4 acc[NS][NTT], sum_of[NS][NTT];  // the chain being summed, the chains before it
    const int m0 = (lane >> 4) * 4;       // first of this lane's 4 rows in a strip
    uint2 res[NS][NTT];              // residual values of this lane's elements, requested ahead of the stream
    if (EPI == EPI_RESID) {
#pragma unroll
      for (int i = 0; i < NS; ++i)
#pragma unroll
        for (int t = 0; t < NTT; ++t) {
          const int col = tok0 + t * 16 + lc;
          res[i][t] = *reinterpret_cast<const uint2*>((const uint16_t*)a.resid + (long long)(col < ntok ? col : ntok - 1) * a.ldo + (strip + i) * 16 + m0);
        }
    }
#pragma unroll
    for (int s = 0; s < NST; ++s) {
      const int kn = s * KC + KC <= NKB ? KC : NKB - s * KC;
      if (s + D < NST) fetch(s + D);
      const u32x4* sx = s_x + (s & 1) * NT * KC * 64 + (kLines ? 0 : lane);
      constexpr bool kOneSet = CH < NKB && NTT > 4;
      constexpr int NB = kOneSet ? 1 : 2;
      u32x4 b[NB][NTT];
#pragma unroll
      for (int t = 0; t < NTT; ++t) b[0][t] = sx[t * KC * 64 + lget(0)];
#pragma unroll
      for (int jj = 0; jj < kn; ++jj) {
        const int j = s * KC + jj;
        if (!kOneSet && jj + 1 < kn) {
#pragma unroll
          for (int t = 0; t < NTT; ++t) b[(jj + 1) % NB][t] = sx[(t * KC + jj + 1) * 64 + lget(jj + 1)];
        }
#pragma unroll
        for (int t = 0; t < NTT; ++t) {
#pragma unroll
          for (int i = 0; i < NS; ++i) {
            if (j % CH == 0 && j > 0) {
              sum_of[i][t] = j == CH ? acc[i][t] : sum_of[i][t] + acc[i][t];
              asm volatile("" : "+v"(sum_of[i][t]));  // (added here and not at the end, which would keep every chain in registers)
            }
            acc[i][t] = mfma_block<BF16>(A[i][j % WIN], b[jj % NB][t], j % CH == 0 ? f32x4{0, 0, 0, 0} : acc[i][t]);
          }
          if (kOneSet && jj + 1 < kn) b[0][t] = sx[(t * KC + jj + 1) * 64 + lget(jj + 1)];
        }
        if (j + WIN < NKB) {
#pragma unroll
          for (int i = 0; i < NS; ++i) A[i][j % WIN] = load_w(i, j + WIN);
        }
        __builtin_amdgcn_sched_barrier(0);  // the refills stay right behind their MFMAs: the window stays full
      }
      if (s + 1 < NST) {
        put(s + 1);  // (that buffer's last readers passed the barrier before this stage)
        lds_barrier();
      }
    }
    if (CH < NKB) {
#pragma unroll
      for (int i = 0; i < NS; ++i)
#pragma unroll
        for (int t = 0; t < NTT; ++t) acc[i][t] = sum_of[i][t] + acc[i][t];
    }
#pragma unroll
    for (int t = 0; t < NTT; ++t) {
      const int col = tok0 + t * 16 + lc;
      if (EPI == EPI_SWIGLU) {
        if (valid[t]) {
          f32x4 r4;
#pragma unroll
          for (int q = 0; q < 4; ++q) r4[q] = (acc[0][t][q] / (1.0f + __expf(-acc[0][t][q]))) * acc[NS - 1][t][q];
          store4<BF16>(a.out0, (long long)(p0 + col) * a.ldo + (strip >> 1) * 16 + m0, r4);
        }
        continue;
      }
#pragma unroll
      for (int i = 0; i < NS; ++i) {
        const f32x4 sum = acc[i][t];
        const bool ok = valid[t] && strip + i < a.n_strips;
        if (EPI == EPI_ARGMAX) {
          // best of the strip's 16 rows (lowest row on equal values): this lane's four, then across the lanes of the token
          float bv = sum[0];
          int bi = (strip + i) * 16 + m0;
#pragma unroll
          for (int q = 1; q < 4; ++q)
            if (sum[q] > bv) { bv = sum[q]; bi = (strip + i) * 16 + m0 + q; }
#pragma unroll
          for (int o = 16; o <= 32; o <<= 1) {
            const float ov = __shfl_xor(bv, o);
            const int oi = __shfl_xor(bi, o);
            if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
          }
          if (ok && lane < 16) {
            ((float*)a.out0)[(long long)col * a.ldo + strip + i] = bv;
            ((int*)a.out1)[(long long)col * a.ldo + strip + i] = bi;
          }
        } else if (EPI == EPI_F32 || EPI == EPI_ROWS) {
          if (ok) *reinterpret_cast<f32x4*>((float*)a.out0 + (long long)(p0 + col) * a.ldo + (strip + i) * 16 + m0) = sum;
        } else if (EPI == EPI_RESID) {
          if (ok) {
            const long long o = (long long)col * a.ldo + (strip + i) * 16 + m0;
            const f32x4 r = {__uint_as_float(res[i][t].x << 16), __uint_as_float(res[i][t].x & 0xFFFF0000u),
                             __uint_as_float(res[i][t].y << 16), __uint_as_float(res[i][t].y & 0xFFFF0000u)};
            store4<BF16>(a.out0, o, r + sum);
          }
        } else if (EPI == EPI_QKV) {  // rotate pairs (i, i + D/2), which sit 32 lanes apart
          const int spd = a.D >> 4;  // strips per head
          const int head = (strip + i) / spd, js = strip + i - head * spd;
          const int half = a.D >> 1;
          const int g4 = lane >> 4;
          const int idx = js * 8 + (g4 & 1) * 4;  // index inside the half
          const bool rot = head < a.Hq + a.Hkv;
          const float* cs = a.rope_cs + (long long)(col < ntok ? col : 0) * a.D + idx;
          const f32x4 cv = *reinterpret_cast<const f32x4*>(cs), sv = *reinterpret_cast<const f32x4*>(cs + half);
          f32x4 other, r4;
#pragma unroll
          for (int q = 0; q < 4; ++q) other[q] = __shfl_xor(sum[q], 32);
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const float c1 = rot ? cv[q] : 1.0f, s1 = rot ? sv[q] : 0.0f;
            r4[q] = (g4 < 2) ? (sum[q] * c1 - other[q] * s1) : (sum[q] * c1 + other[q] * s1);
          }
          if (ok) {
            const int hrow = (g4 < 2 ? 0 : half) + idx;
            if (head < a.Hq) store4<BF16>(a.out0, ((long long)col * a.Hq + head) * a.D + hrow, r4);
            else if (head < a.Hq + a.Hkv) store4<BF16>(a.out1, ((long long)col * a.Hkv + (head - a.Hq)) * a.D + hrow, r4);
            else store4<BF16>(a.out2, ((long long)col * a.Hkv + (head - a.Hq - a.Hkv)) * a.D + hrow, r4);
          }
        }
      }
    }
  };
  // the number of live token tiles is known per piece of work: one compiled body for each (for a token group of the layer's
  // projections, where all but the last are full: one for a single tile, one for more)
  constexpr bool kEach = GROUPED || EPI == EPI_ROWS || EPI == EPI_ARGMAX;
  // In step: the token groups of a strip group run side by side and share its weights through L2 as long as neither gets
  // ahead, so the last group of several goes at the pace of the full ones where it has more than half as many tiles (LM head,
  // 151936 x 2048, score rows of 104 tokens: 193 us with 4 and 3 tiles, 184 with 4 and 4).
  auto dispatch = [&](const u32x4* wbase, int sg, int p0, int ntok, int tok0, bool in_step) __attribute__((always_inline)) {
    int live = (ntok - tok0 + 15) >> 4;
    if (in_step && live * 2 > NT) live = NT;
    if (live <= 1) run(std::integral_constant<int, 1>{}, wbase, sg, p0, ntok, tok0);
    else if (kEach && NT >= 3 && live == 2) run(std::integral_constant<int, (kEach && NT >= 3 ? 2 : 1)>{}, wbase, sg, p0, ntok, tok0);
    else if (kEach && NT >= 4 && live == 3) run(std::integral_constant<int, (kEach && NT >= 4 ? 3 : 1)>{}, wbase, sg, p0, ntok, tok0);
    else if (kEach && NT >= 5 && live == 4) run(std::integral_constant<int, (kEach && NT >= 5 ? 4 : 1)>{}, wbase, sg, p0, ntok, tok0);
    else run(std::integral_constant<int, NT>{}, wbase, sg, p0, ntok, tok0);
  };

  if (GROUPED) {
    const int total = *a.union_count * nsg;
    for (int chunk = blockIdx.x; chunk < total; chunk += gridDim.x) {
      const int slot = chunk / nsg;
      const WorkRec* rec = a.work + slot;
      const int ex = rec->expert;
      const u32x4* wbase = ex < a.n_routed ? a.W + (long long)ex * a.group_stride
                                           : a.W_shared + (long long)(ex - a.n_routed) * a.group_stride;
      dispatch(wbase, chunk - slot * nsg, rec->p0, rec->ntok, 0, false);
    }
  } else {
    // workgroup ids go round-robin over the 8 XCDs: the token groups of a strip group are 8 apart and share an L2
    const int T = dyn_tokens(a.T_dev, a.T);
    const unsigned ntg = (unsigned)a.dense_tiles;
    const unsigned xcd = blockIdx.x & 7u, q = blockIdx.x >> 3;
    const unsigned tg = q % ntg, sg = (q / ntg) * 8u + xcd;
    if (sg >= (unsigned)nsg || (int)tg * NT * 16 >= T) return;  // (whole workgroup, before any barrier)
    const int tok0 = (int)tg * NT * 16;
    dispatch(a.W, (int)sg, 0, T < tok0 + NT * 16 ? T : tok0 + NT * 16, tok0, T > NT * 16);
  }
}

}  // namespace evict
