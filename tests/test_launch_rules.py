"""The rules that choose kernels by size and by the launch-shape knobs (csrc/launch_rules.h), compiled for the host."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CXX = shutil.which("g++")
SHIM = """
#include "launch_rules.h"
using namespace evict;
extern "C" {
int moe_auto(const int* k) {
  return moe_knobs_auto(MoeKnobs{k[0], k[1], k[2], k[3], k[4], k[5], k[6], k[7], k[8], k[9]});
}
int dense_auto(int kernel, int nt, int ntw, int units, int nt_loads) { return dense_knobs_auto(kernel, nt, ntw, units, nt_loads); }
int chunk(int slots, int pairs) { return gateup_chunk(slots, gateup_chunk_counts(pairs)); }
int tiled(int T, int k, int E, int nkb, int pairs, int strip) { return experts_tiled(T, k, E, nkb, pairs, strip); }
int lm(int T, int n_strips, int nkb) { return lm_tiled(T, n_strips, nkb); }
int units(int T, int n_strips) { return lm_units(T, n_strips); }
int strips(int T, int n_strips) { return lm_strips(T, n_strips); }
int one_round(int T, int n_strips, int nkb, int bf16) { return lm_one_round(T, n_strips, nkb, bf16); }
int deal(int T, int n_strips, int nkb, int bf16) { return lm_deal(T, n_strips, nkb, bf16); }
int keeps_best(int n_strips, int nkb, int bf16) { return lm_keeps_best(n_strips, nkb, bf16); }
int keeps_rows(int T, int n_strips, int nkb, int bf16) { return lm_keeps_rows(T, n_strips, nkb, bf16); }
int topk(int T, int E, int k) { return topk_by_rows(T, E, k); }
int grid(int n_strips, int strips, int groups) { return tile_grid(n_strips, strips, groups); }
int rows_applies(int D, int B, int T, int Hq, int Hkv, int ctx) { return attn_rows_applies(D, B, T, Hq, Hkv, ctx); }
int rows_one_tree(int T, int Hq, int Hkv, int ctx) { return attn_rows_one_tree(T, Hq, Hkv, ctx); }
int rows_splits(int wgs, int Hkv, int rbs) { return attn_rows_splits(wgs, Hkv, rbs); }
int rows_strides(int B, long long seq, long long head) { return attn_rows_strides(B, seq, head); }
int rows_wgs(int B, int T, int Hq, int Hkv, int ctx) { return attn_rows_wgs(B, T, Hq, Hkv, ctx); }
int down_nt(int knob, int nkb) { return down_nt_loads(knob, nkb); }
}
"""
pytestmark = pytest.mark.skipif(CXX is None, reason="no host compiler")


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "shim.cpp").write_text(SHIM)
    so = str(d / "rules.so")
    subprocess.run([CXX, "-std=c++17", "-Wall", "-Werror", "-Wno-unknown-pragmas", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_2605_00342_amd", "csrc"),
                    "-o", so, str(d / "shim.cpp")], check=True)
    return ctypes.CDLL(so)


# nt, gateup_kernel, down_kernel, pair_down, down_ws, nt_loads, lds_dma, prefetch, chunk_gateup, chunk_down as evict_create sets them
DEFAULTS = dict(nt=0, gateup_kernel=2, down_kernel=1, pair_down=2, down_ws=0, nt_loads=2, lds_dma=1, prefetch=1, chunk_gateup=0, chunk_down=0)


def moe_auto(rules, **knobs):
    k = dict(DEFAULTS, **knobs)
    return bool(rules.moe_auto((ctypes.c_int * 10)(*k.values())))


def test_expert_knobs_ask_for_their_kernels(rules):
    assert moe_auto(rules) and moe_auto(rules, nt_loads=1)
    for name, values in (("nt", (1, 2)), ("gateup_kernel", (0, 1)), ("down_kernel", (0,)), ("pair_down", (0, 1)), ("down_ws", (8, 16)),
                         ("nt_loads", (0,)), ("lds_dma", (0,)), ("prefetch", (3,)), ("chunk_gateup", (1, 2, 4)), ("chunk_down", (1, 4))):
        for v in values:
            assert not moe_auto(rules, **{name: v}), (name, v)


def test_projection_knobs_ask_for_their_kernels(rules):
    assert rules.dense_auto(2, 0, 0, 0, 2) and rules.dense_auto(2, 0, 0, 0, 1)
    for args in ((0, 0, 0, 0, 2), (1, 0, 0, 0, 2), (2, 1, 0, 0, 2), (2, 0, 1, 0, 2), (2, 0, 0, 4, 2), (2, 0, 0, 0, 0)):
        assert not rules.dense_auto(*args), args


def test_down_loads_follow_the_knob(rules):
    for nkb in (6, 8, 24, 44):
        assert rules.down_nt(0, nkb) == 0 and rules.down_nt(1, nkb) == 1
    assert [rules.down_nt(2, n) for n in (6, 8, 24, 44)] == [1, 0, 1, 1]


def test_gateup_chunk(rules):
    for pairs in (1, 3, 5, 12, 16, 24, 32, 96):
        for slots in (0, 1, 2, 21, 22, 43, 46, 64, 66, 130, 300, 8192 + 1024):
            c = rules.chunk(slots, pairs)
            assert 1 <= c <= 4 and pairs % c == 0
            if 0 < slots * pairs <= 256:
                assert c == 1  # all in one round already
    # measured the best, or within 2 % of it
    assert [rules.chunk(s, 12) for s in (17, 22, 43, 46, 66)] == [1, 2, 3, 3, 4]
    assert [rules.chunk(57, 12), rules.chunk(35, 16), rules.chunk(36, 16)] == [3, 4, 4]
    assert [rules.chunk(s, 16) for s in (64, 69, 130, 144, 300)] == [2] * 5  # two full rounds of two pairs and more


def test_tiled_experts(rules):
    # (T, k, E, blocks, strip pairs, strip kernels' size)
    assert rules.tiled(96, 8, 128, 64, 48, 1) and not rules.tiled(95, 8, 128, 64, 48, 1)   # 6 tokens per expert
    assert rules.tiled(86, 6, 64, 64, 88, 1) and not rules.tiled(85, 6, 64, 64, 88, 1)     # 8: 88 pairs are no multiple of 6
    assert rules.tiled(160, 8, 128, 128, 12, 1) and not rules.tiled(159, 8, 128, 128, 12, 1)
    assert rules.tiled(320, 8, 256, 128, 16, 0)                                            # (no strip kernel of 128 blocks)
    assert not rules.tiled(63, 8, 64, 64, 48, 0)                                           # the contraction split's sums
    assert not rules.tiled(512, 4, 16, 64, 16, 1) and not rules.tiled(512, 4, 16, 64, 48, 1)  # too few workgroups


def test_tile_grid(rules):
    assert rules.grid(320, 4, 3) == 240 and rules.grid(128, 8, 4) == 64
    assert rules.grid(160, 8, 12) == 288 and rules.grid(160, 8, 10) == 240 and rules.grid(1, 8, 1) == 8
    for n_strips in (1, 7, 80, 128, 160, 320, 384, 9496):
        for strips in (4, 8, 16):
            for groups in (1, 2, 11):
                wgs = rules.grid(n_strips, strips, groups)
                # the fullest XCD's share of the grid, eight times
                assert wgs == 8 * groups * -(-(-(-n_strips // strips)) // 8)


def test_lm_head(rules):
    big = 9496
    assert [rules.lm(T, big, 64) for T in (16, 32, 33, 128)] == [0, 0, 1, 1]
    assert [rules.lm(T, big, 128) for T in (8, 11, 12, 16, 128)] == [0, 0, 1, 1, 1]
    assert not rules.lm(96, 1000, 64) and rules.lm(96, 2000, 64)          # few strips: too few workgroups
    assert not rules.lm(16, 512, 128) and rules.lm(16, 1000, 128) and rules.lm(17, 64, 128)
    assert not rules.lm(96, 2001, 64) and not rules.lm(96, 2000, 32)      # odd strip counts, lengths that are not built
    assert [rules.units(T, big) for T in (1, 9, 12, 13, 16, 17)] == [2, 2, 2, 8, 8, 8]
    assert rules.units(16, 1000) == 2 and rules.units(32, 64) == 8


def test_lm_head_rounds(rules):
    assert [rules.strips(T, 9496) for T in (1, 13, 16, 17, 32)] == [2, 8, 8, 38, 38]
    for n in (64, 1024, 2048, 2049, 6400, 9496, 12504):
        s = rules.strips(32, n)
        assert s >= 8 and -(-n // s) <= 256


def test_lm_head_rounds_where_they_were_measured_faster(rules):
    for T in (17, 24, 32):
        assert rules.one_round(T, 9496, 32, 1) and rules.one_round(T, 9496, 48, 1) and rules.one_round(T, 6400, 64, 1)
        assert bool(rules.one_round(T, 9496, 64, 1)) == (T > 24)
        # slower, or not faster: 32 strips of 96 blocks each, 9 of 128; 32-bit storage
        assert not (rules.one_round(T, 8016, 96, 1) or rules.one_round(T, 2049, 128, 1) or rules.one_round(T, 4096, 64, 0))
    assert rules.one_round(96, 9496, 32, 1) and not rules.one_round(33, 4097, 64, 1)  # several groups of 32 tokens


def test_topk_rows_where_they_were_measured_faster(rules):
    for E, k, first in ((16, 2, 17), (64, 6, 17), (128, 8, 17), (128, 1, 17), (64, 16, 17), (144, 4, 28), (256, 8, 28), (256, 16, 28)):
        assert [T for T in range(1, 33) if rules.topk(T, E, k)] == list(range(first, 33))
    assert not any(rules.topk(T, 64, 17) for T in range(1, 33))  # (a row of 16 lanes has no room for 17 picks)


def test_attention_rows(rules):
    f = rules.rows_applies
    assert not f(64, 16, 256, 32, 4, 6000) and not f(128, 65, 520, 32, 4, 2048)  # other head dimension, too many sequences
    assert f(128, 1, 8, 32, 4, 0) and f(128, 1, 64, 16, 16, 1 << 20) and f(128, 16, 16, 8, 1, 0) and f(128, 64, 64, 8, 1, 100)
    assert not f(128, 1, 9, 32, 4, 100) and not f(128, 15, 120, 32, 4, 100)
    edge = [L for L in range(64, 8192, 64) if f(128, 1, 64, 32, 4, L)][0]  # 4 row blocks x 4 heads x (chunks + 1)
    assert edge == 24 * 64 and not f(128, 1, 64, 32, 4, edge - 64) and f(128, 1, 64, 32, 4, edge - 63)
    assert rules.rows_wgs(16, 900, 32, 4, 2048) == 512 and rules.rows_wgs(1, 128, 32, 4, 4096) == 256


def test_lm_head_deal(rules):
    assert [rules.deal(T, 9496, 64, 1) for T in (1, 12, 13, 16, 17, 24, 32)] == [2, 2, 38, 38, 38, 38, 38]
    assert rules.deal(16, 4096, 64, 1) == 8 and rules.deal(16, 4097, 64, 1) == 17 and rules.deal(16, 9729, 64, 1) == 8  # 39 strips: past the line
    for T, n, nkb, bf16 in ((16, 9496, 32, 1), (24, 9496, 128, 1), (24, 9496, 64, 0), (8, 9496, 64, 1), (48, 9496, 48, 1)):
        old = rules.strips(T, n) if rules.one_round(T, n, nkb, bf16) else rules.units(T, n)
        assert rules.deal(T, n, nkb, bf16) == old


def test_attention_rows_need_aligned_rows(rules):
    def f(B, seq, head):
        return bool(rules.rows_strides(B, ctypes.c_longlong(seq), ctypes.c_longlong(head)))

    assert f(1, 0, 128 * 100) and f(4, 128 * 400, 128 * 100) and f(4, 128 * 400 + 8, 128 * 100 + 8) and f(1, 3, 8)
    for off in (1, 2, 4, 7):
        assert not f(1, 0, 128 * 100 + off) and not f(2, 128 * 400 + off, 128 * 100) and not f(2, 128 * 400, 128 * 100 + off)
    assert not f(1, 0, (1 << 33) + 4) and f(1, 0, (1 << 33) + 8)


def test_lm_head_keeps_results_only_of_many_strips(rules):
    """Where a workgroup has few strips, what it would keep is stored strip by strip, as it is where the kept form is not built."""
    for nkb in (64, 128, 192):
        assert [rules.keeps_best(n, nkb, 1) for n in (1, 64, 1000, 2048, 2049, 9496)] == [0, 0, 0, 0, 1, 1]
        assert [rules.keeps_rows(13, n, nkb, 1) for n in (1, 64, 1000, 2048, 2049, 9496)] == [0, 0, 0, 0, 1, 1]
    assert [rules.keeps_best(n, 24, 1) for n in (64, 1536, 1537)] == [0, 0, 1]
    assert rules.keeps_rows(1, 9496, 64, 1) and not rules.keeps_rows(12, 9496, 128, 1)
    for nkb in (8, 16, 24, 32, 48, 96):
        assert not rules.keeps_rows(32, 9496, nkb, 1) and (nkb == 24 or not rules.keeps_best(9496, nkb, 1))
    assert not rules.keeps_best(9496, 64, 0) and not rules.keeps_rows(32, 9496, 64, 0)


def test_attention_splits_leave_no_xcd_a_second_round(rules):
    for wgs in (256, 512):
        for Hkv in (1, 2, 4, 8, 16, 32):
            for rbs in range(1, 65):
                n = rules.rows_splits(wgs, Hkv, rbs)
                assert n >= 1
                if n > 1:
                    assert (n * Hkv + 7) // 8 * rbs <= wgs // 8, (wgs, Hkv, rbs, n)
    assert [rules.rows_splits(256, 4, r) for r in (1, 2, 3, 4, 7, 8)] == [64, 32, 20, 16, 8, 8]


def test_attention_rows_where_they_were_measured_faster(rules):
    """Batches of few rows, which lie within one workgroup of the 16-row kernel per KV head, and large trees of one or two KV heads."""
    f = rules.rows_applies
    for ctx, want in ((600, 0), (1000, 0), (3000, 0), (4096, 1), (10000, 1)):  # 4 trees of 8 nodes, 16 heads of one: 64 units
        assert bool(f(128, 4, 32, 16, 16, ctx)) == bool(want), ctx
    assert [bool(f(128, 8, 8, 16, 16, c)) for c in (100, 1000, 1984, 2048)] == [False, False, True, True]
    assert [bool(f(128, 12, 12, 16, 16, c)) for c in (100, 300, 384, 600)] == [False, False, True, True]  # 192 units
    assert f(128, 20, 20, 16, 16, 100) and not f(128, 16, 16, 16, 16, 100)  # 320 units and 256
    assert [bool(f(128, 8, 8, 32, 4, c)) for c in (600, 2048, 6000)] == [False, False, False] and f(128, 9, 9, 32, 4, 6000)
    for shape, lo, hi in (((2, 187, 8, 1), 3000, 5000), ((3, 369, 8, 1), 2048, 4000), ((1, 64, 16, 2), 6000, 8192), ((1, 48, 64, 8), 2048, 3000),
                          ((2, 187, 16, 16), 1500, 2048)):
        assert not f(128, *shape, lo) and f(128, *shape, hi), shape
    assert f(128, 1, 44, 8, 1, 15161) and f(128, 1, 64, 8, 1, 8193) and not f(128, 1, 64, 8, 1, 8192)  # long contexts
    assert f(128, 1, 100, 16, 16, 1600) and f(128, 2, 120, 32, 4, 1500) and f(128, 5, 360, 8, 1, 2000)


def test_attention_rows_of_one_tree(rules):
    """From 12 chunks of 64 keys per CU on, the draft nodes' chunk among them; where the general rule takes the kernel too."""
    f = rules.rows_one_tree
    assert [bool(f(128, 32, 4, c)) for c in (4096, 6016, 6017, 32000)] == [False, False, True, True]  # 8 row blocks x 4 heads x (chunks + 1)
    assert [bool(f(n, 32, 32, 6100)) for n in (1, 64, 128)] == [True, True, True] and not f(64, 16, 16, 8192) and not f(1, 32, 4, 32768)
    for shape in ((128, 32, 4, 6017), (100, 16, 2, 14100), (1, 32, 32, 6100), (64, 64, 8, 6017), (128, 8, 1, 24513)):
        assert f(*shape) and rules.rows_applies(128, 1, *shape)
