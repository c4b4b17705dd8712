"""Index, plan and routing arithmetic of the launches (csrc/launch_math.h), compiled with the host compiler and checked at sizes
that no GPU test launches."""
import ctypes as C
import os
import shutil
import subprocess

import pytest

from tile_cases import QKV_SEAMS, QKV_TILES, ROPE_TILES, SEAMS, SLICED_ALONE, SLICED_DIMS, SLICED_ROWS, TILES

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = r"""
#include "launch_math.h"
extern "C" {
unsigned clear_blocks() { return fv::kClearBlocks; }
unsigned clear_threads() { return fv::kClearThreads; }
int clears(unsigned block) { return fv::clears_counters(block); }
void share(unsigned block, unsigned thread, unsigned blocks, int* out) {
    const fv::CounterShare s = fv::counter_share(block, thread, blocks);
    out[0] = s.first;
    out[1] = s.step;
}
void plan(int N, int K, int layernorm, int* out) {
    const fv::FewRowsPlan p = fv::few_rows_plan(N, K, layernorm);
    out[0] = p.cols;
    out[1] = p.waves;
    out[2] = p.turns;
    out[3] = fv::few_rows_share(K, p.cols);
}
int few_rows(int M, int N, int K, int split_k) { return fv::few_rows_product(M, N, K, split_k); }
int xcd_share(int block, int n, int runs, int sample) { return fv::xcd_share(block, n, runs, sample); }
int xcd_blocks(int n, int runs) { return fv::xcd_blocks(n, runs); }
int in_runs(int n, int w, int rows) { return fv::shares_in_runs(n, w, rows); }
int column_chunks(int N, int D) { return fv::column_chunks(N, D); }
void prefetch(const long* bytes, int n, int idle, double us, int cut, long* out) {
    const fv::PrefetchPlan p = fv::prefetch_plan(bytes, n, idle, us, cut);
    out[0] = p.bytes;
    out[1] = p.blocks;
}
int tile(int qkv, int M, int N, int K) { return fv::gemm_choose_tile(qkv, M, N, K).cfg; }
long slices(int M, int N, int K, int meet, int* out) {
    const fv::SplitKPlan p = fv::gemm_splitk_plan(M, N, K, static_cast<fv::SlicesMeet>(meet));
    out[0] = p.cfg;
    out[1] = p.splits;
    return (long)p.bytes;
}
int restore_rows(long rows, int w, int D) {
    const fv::RestorePlan p = fv::restore_plan(rows, w, D);
    return p.pair ? -p.rows : p.rows;
}
void ahead(int D, int F, int M, int in_stack, int ffn_follows, long* out) {
    const fv::AheadList l = fv::ahead_list(D, F, M, in_stack, ffn_follows);
    out[0] = l.n;
    for (int i = 0; i < 3; ++i) out[1 + i] = l.bytes[i];
}
int attention(int B, int H, int dh, int k, int L) { return fv::attention_cfg(B, H, dh, k, L); }
int attention_slices(int B, int H, int k, int L) {
    const fv::AttentionSlices s = fv::attention_slices(B, H, k, L);
    return s.queries * 10 + s.slices;
}
int wide_stages_a(int bm, int bn, int bk, int stages) { return fv::wide_stages_a(bm, bn, bk, stages); }
int load_slots(int slots, int before, int ksteps, int loads) { return fv::load_slots(slots, before, ksteps, loads); }
int handover_loads(int slots, int before, int ls, int loads) { return fv::handover_loads(slots, before, ls, loads); }
int out_at_start(int sa, int stages, int a_ld, int w_ld, int window) { return fv::wide_out_at_start(sa, stages, a_ld, w_ld, window); }
int out_at_handover(int sa, int stages, int a_ld, int w_ld, int left) { return fv::wide_out_at_handover(sa, stages, a_ld, w_ld, left); }
int few_rows_in_lds(int M, int N, int K, int layernorm) { return fv::few_rows_in_lds(M, N, K, layernorm); }
int few_rows_ln(int M, int N, int K) { return fv::few_rows_layernorm(M, N, K); }
}
"""


@pytest.fixture(scope="module")
def math(tmp_path_factory):
    cxx = shutil.which("g++") or "/opt/rocm/bin/amdclang++"
    d = tmp_path_factory.mktemp("launch_math")
    src, so = d / "shim.cpp", d / "shim.so"
    src.write_text(SHIM)
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2503_23367_amd", "csrc"), "-o", str(so), str(src)], check=True)
    return C.CDLL(str(so))


def _share(math, block, thread, blocks):
    out = (C.c_int * 2)()
    math.share(C.c_uint(block), C.c_uint(thread), C.c_uint(blocks), out)
    return out[0], out[1]


@pytest.mark.parametrize("blocks", [1, 2, 255, 256, 257, 1 << 23, (1 << 23) + 1, 1 << 24, (1 << 31) - 1])
def test_counter_shares_stay_in_range_and_cover_every_counter_once(math, blocks):
    """A flat index over all workgroups passes 2^31 at 2^23 workgroups of 256 threads, turns negative, and a thread of a
    launch without any counters then stores through the null pointer."""
    threads, most = math.clear_threads(), math.clear_blocks()
    for block in {0, 1, most - 1, most, min(blocks, 1 << 23), (1 << 23) - 1, (1 << 23) + 5, blocks - 1}:
        if not 0 <= block < blocks or not math.clears(C.c_uint(block)):
            continue
        for thread in (0, 1, threads - 1):
            first, step = _share(math, block, thread, blocks)
            assert 0 <= first < step <= most * threads, (block, thread)
    for n in (0, 1, 300, 70000):
        seen = [0] * n
        for block in range(min(blocks, most + 2)):
            if math.clears(C.c_uint(block)):
                for thread in range(threads):
                    first, step = _share(math, block, thread, blocks)
                    for i in range(first, n, step):
                        seen[i] += 1
                    if first >= n:
                        break
        assert seen == [1] * n


@pytest.mark.parametrize("layernorm", [0, 1])
@pytest.mark.parametrize("N", [64, 2048, 2304, 4096, 4104, 24576])
def test_few_rows_turns_past_the_end_are_less_than_one_a_wave_and_round(math, N, layernorm):
    """A wave whose turns are used up loads the last one again: four turns in flight for every K loaded 64 for 18."""
    for K in range(64, 33000, 64):
        out = (C.c_int * 4)()
        math.plan(N, K, layernorm, out)
        cols, waves, turns, share = out
        assert (cols, waves) in ((16, 8), (8, 8), (8, 16)) and 1 <= turns <= 4 and share == -(-K // (64 * (16 // cols)))
        if layernorm and K <= 2048:
            assert cols == 16 and waves == 8 and waves * turns >= share   # the rows of a wave's whole share stay in registers
        rounds = -(-share // (waves * turns))
        assert rounds * waves * turns - share < rounds * waves, (K, waves, turns)


# Shapes whose few-row product was measured slower than the tiled one (M, N, K, the tiled one splits K).
TILED = [(16, 32768, 1024, 0), (8, 24576, 1024, 0), (16, 65536, 512, 0), (16, 16384, 2048, 0), (8, 16384, 2304, 0),
         (16, 2304, 9216, 1), (1, 2304, 9216, 1), (1, 2176, 2176, 1), (12, 24576, 8192, 0), (16, 32768, 8192, 0),
         (16, 1920, 7680, 1), (2, 5120, 20480, 1), (17, 64, 64, 0)]
# ... and faster.
FEW = [(1, 6144, 2048, 1), (16, 6144, 2048, 1), (16, 8192, 2048, 0), (1, 2048, 8192, 1), (8, 1920, 7680, 1),
       (16, 1024, 4096, 1), (16, 12288, 4096, 0), (8, 16384, 4096, 0), (1, 32768, 8192, 0), (16, 64, 64, 0),
       (16, 256, 16384, 0), (16, 4096, 1024, 0)]


def test_few_rows_through_lds(math):
    """Rows that fit go through LDS whatever the number of workgroups; one row over exactly a round of K, on as many workgroups a CU, was 3
    to 6 % slower that way (16384 x 2048 13.8 us, 13.3 without)."""
    for M, N, K, layernorm in [(1, 2048, 8192, 0), (16, 12288, 4096, 1), (8, 24576, 2048, 1), (2, 16384, 2048, 1), (1, 6144, 2048, 1), (1, 12288, 1984, 1),
                               (1, 12288, 4096, 1), (1, 12288, 2048, 0), (1, 2048, 2048, 0)]:
        assert math.few_rows_in_lds(M, N, K, layernorm), (M, N, K)
    for M, N, K, layernorm in [(1, 4096, 2048, 1), (1, 16384, 2048, 1), (1, 24576, 2048, 1), (9, 2048, 8192, 0), (5, 4096, 16384, 0)]:
        assert not math.few_rows_in_lds(M, N, K, layernorm), (M, N, K)


def test_few_rows_routing(math):
    for case in TILED:
        assert not math.few_rows(*case), case
    for case in FEW:
        assert math.few_rows(*case), case
    # A block whose shapes have no split-K scratch asks without it: what the scratch's plan gave to the few-row product
    # has to go there then too.
    for M in range(1, 18):
        for N in range(64, 8193, 64):
            for K in (64, 1024, 2048, 2112, 2304, 3072, 4096, 4352, 6144, 8192, 9216, 16384, 20480, 32768):
                assert not math.few_rows(M, N, K, 1) or math.few_rows(M, N, K, 0), (M, N, K)
                assert not math.few_rows_ln(M, N, K) or K <= 2048 and math.few_rows(M, N, K, 1), (M, N, K)


def test_tile_cases_reach_their_tiles(math):
    for cfg, cases in TILES.items():
        for M, N, K, _ in cases:
            assert math.tile(0, M, N, K) == cfg, (M, N, K)
    for cfg, (D, _, B, k) in [*QKV_TILES.items(), *QKV_SEAMS.items(), *ROPE_TILES.items()]:
        assert math.tile(1, B * k, 3 * D, D) == cfg, (B, k, D)
    # a workgroup takes a second tile from 257 tiles on (one workgroup a CU)
    sizes = {11: (256, 256), 38: (224, 256), 12: (256, 192), 37: (224, 192), 14: (192, 192), 13: (192, 256), 32: (256, 128)}
    for cfg, cases in SEAMS.items():
        for M, N, K, _ in cases:
            assert math.tile(0, M, N, K) == cfg and -(-M // sizes[cfg][0]) * -(-N // sizes[cfg][1]) > 256, (M, N, K)
    for cfg, (D, _, B, k) in QKV_SEAMS.items():
        assert -(-B * k // sizes[cfg][0]) * -(-3 * D // sizes[cfg][1]) > 256, (B, k, D)


# (qkv, M, N, K): a tile that is 3 to 50 % slower there than the one picked, us
SLOWER = [((0, 320, 6336, 192), 13), ((0, 1462, 4224, 640), 13),                       # 11.2 / 5.6, 19.2 / 15.0
          ((0, 3309, 4096, 16384), 35), ((0, 787, 4096, 16384), 35), ((0, 10418, 2560, 8192), 34),   # 399 / 314, 158 / 117, 429 / 328
          ((1, 4242, 6912, 2304), 34), ((1, 1095, 7680, 2560), 34),                    # 152 / 116, 64 / 43
          ((0, 391, 256, 128), 18), ((0, 284, 1216, 192), 18),                         # 4.40 / 4.02, 4.23 / 4.11
          ((1, 68, 5760, 1920), 16), ((1, 76, 6144, 2048), 16)]                        # 11.9 / 10.7, 12.0 / 10.7


def test_tiles_are_not_the_ones_measured_slower(math):
    for shape, cfg in SLOWER:
        assert math.tile(*shape) != cfg, shape
    # where 64x32 tiles are at most a round and K is long enough for their two k-groups, and just past either
    for M, N, K, cfg in [(64, 8192, 320, 18), (64, 8192, 256, 16), (128, 4096, 1024, 18), (128, 4104, 1024, 16), (129, 8192, 1024, 17)]:
        assert math.tile(0, M, N, K) == cfg, (M, N, K)
    # every size has a tile that the launch knows
    for M in (17, 64, 65, 191, 193, 1000, 4097, 33000, 87381):
        for N in (8, 64, 1344, 6144, 24576, 32768):
            for K in (64, 448, 2048, 2112, 8192, 32768):
                assert math.tile(0, M, N, K) in TILES and math.tile(1, M, N, K) in {15, *TILES}, (M, N, K)


# tiles on four waves, one a SIMD (rows, columns, stages of W), those of other rings that one may want, and rings of two
WIDE = [(256, 256, 3), (256, 192, 3), (224, 256, 3), (224, 192, 3), (224, 128, 3), (192, 256, 3), (192, 192, 3), (160, 128, 4),
        (128, 128, 3), (128, 128, 4), (128, 128, 5), (128, 64, 6), (192, 192, 2), (256, 128, 3)]


@pytest.mark.parametrize("bm,bn,stages", WIDE)
def test_wide_tiles_wait_for_the_next_tile_and_no_more(math, bm, bn, stages):
    """The main loop's order of loads, replayed: at every hand-over the loads that may still be out are those behind the next tile's last
    one.  With four stages it once waited as with three, and the fourth bought nothing."""
    sa = math.wide_stages_a(bm, bn, 64, stages)
    a_ld, w_ld, ksteps = bm // 32, bn // 32, 2
    slots, loads = (bm // 32) * (bn // 32), a_ld + w_ld
    before = 4 if slots >= 32 else 2
    every = math.load_slots(slots, before, ksteps, loads)
    assert every > 0 and (stages - 1) * loads <= 63
    first = math.handover_loads(slots, before, every, loads)
    for tiles in list(range(1, 12)) + [32]:
        order = []   # (operand, K tile) of every load, as issued

        def window(a_tile, w_tile, lo, hi):
            for q in range(lo, hi):
                operand, tile = ("A", a_tile) if q < a_ld else ("W", w_tile)
                if tile < tiles:
                    order.append((operand, tile))

        def check(tile, out):
            last = max(i for i, (_, t) in enumerate(order) if t == tile)
            assert {(o, t) for o, t in order if t == tile} == {("A", tile), ("W", tile)}
            assert [order.count((o, tile)) for o in "AW"] == [a_ld, w_ld]
            assert out == len(order) - 1 - last, (tiles, tile, out, order[last:])

        for s in range(min(stages - 1, tiles)):
            if s < sa - 1:
                order += [("A", s)] * a_ld
            order += [("W", s)] * w_ld
        window(sa - 1, stages - 1, 0, first)
        if tiles >= stages:
            check(0, math.out_at_start(sa, stages, a_ld, w_ld, first))
        for kt in range(tiles - 1):
            # the rest of the window that the hand-over in front opened: in this tile's k-steps but the last
            in_steps = sum(1 for i in range((ksteps - 1) * slots) if i % every == every // 2)
            assert first + in_steps >= loads
            window(kt + sa - 1, kt + stages - 1, first, loads)
            check(kt + 1, math.out_at_handover(sa, stages, a_ld, w_ld, tiles - 1 - kt))
            window(kt + sa, kt + stages, 0, first)


LAYERNORM, EITHER, LAUNCH = 0, 1, 2   # SlicesMeet


def _slices(math, M, N, K, meet):
    out = (C.c_int * 2)()
    math.slices.restype = C.c_long
    size = math.slices(M, N, K, meet, out)
    return size, out[0], out[1]


def test_slices_of_a_half_pay_for_their_own_launch(math):
    """No LayerNorm follows the out-proj of an attention half on its own.  Cut there all the same, as in a whole block, its calls were 3 to
    11 % slower than whole (us, cut / whole): 357 rows 2304 wide 56.1 / 51.0, 479 and 443 of the small model 30.5 / 27.4, 30.1 / 27.1,
    226 of 1920 34.3 / 32.3, 271 of 2048 42.4 / 39.7."""
    for M, D in [(357, 2304), (479, 1024), (443, 1024), (226, 1920), (190, 1920), (271, 2048), (254, 2048), (201, 1024)]:
        assert _slices(math, M, D, D, LAUNCH)[2] == 1, (M, D)
    # ... and seven tile rows of 128 or 160 in two slices (MLP half of 813 rows 82.9 / 78.8, 974 of 9216: 131 / 118)
    for M, N, K in [(813, 1920, 7680), (825, 1920, 7680), (974, 2304, 9216), (1328, 2304, 9216)]:
        _, cfg, splits = _slices(math, M, N, K, LAUNCH)
        rows = {40: 128, 35: 160, 34: 192}.get(cfg, 64)
        assert splits == 1 or -(-M // rows) != 7, (M, N, K, cfg, splits)
    # where slices win by several us they are kept: MLP half of 545 / 395 rows 67.7 / 62.4, 60.1 / 49.5
    for M, N, K in [(64, 2048, 8192), (256, 2048, 8192), (576, 2048, 8192), (395, 1920, 7680), (545, 1920, 7680)]:
        assert _slices(math, M, N, K, LAUNCH)[2] > 1 and _slices(math, M, N, K, EITHER)[2] > 1, (M, N, K)


def test_slices_of_a_block_where_whole_small_tiles_are_slower(math):
    """Out-proj inside a block, whose LayerNorm adds the slices up: whole, on 64x64 and 128x64 tiles that the model had a microsecond too
    fast, stacks of 294 rows were 1.5 % slower (1920 wide 761 us for eight blocks, 749 in two slices; 2304 wide 890 / 874)."""
    for M, D in [(259, 1920), (286, 1920), (294, 1920), (400, 1920), (294, 2304), (446, 2304)]:
        assert _slices(math, M, D, D, LAYERNORM)[2] == 2, (M, D)
    # ... but on their own the launch that adds up costs more than that (MLP half, slices / whole: 683 and 676 rows 2304 wide 73.8 / 65.9, 73.5 / 66.7)
    for M, N, K in [(683, 2304, 6912), (676, 2304, 6912), (286, 1920, 1920)]:
        assert _slices(math, M, N, K, LAUNCH)[2] == 1, (M, N, K)


def test_slices_fit_their_launch(math):
    """At most a round of workgroups, whole K tiles in every slice, tiles and counts that the launches know, and scratch for them all."""
    for M in list(range(1, 140)) + [191, 256, 257, 400, 576, 731, 960, 1152, 2241, 4096, 70000]:
        for N, K in [(64, 64), (448, 2048), (1024, 1024), (1024, 4096), (1920, 7680), (2048, 8192), (2176, 2176), (2304, 9216), (8192, 32768)]:
            for meet in (LAYERNORM, EITHER, LAUNCH):
                size, cfg, splits = _slices(math, M, N, K, meet)
                if splits == 1:
                    assert size == 0
                    continue
                bm, bn = {16: (64, 64), 17: (128, 64), 40: (128, 128), 35: (160, 128), 34: (192, 128)}[cfg]
                assert splits in (2, 4, 8) and K // 64 % splits == 0 and size == 4 * splits * M * N
                assert -(-M // bm) * -(-N // bn) * splits <= 256
                assert not math.few_rows(M, N, K, 1) or not (K >= 2048 and K // 64 % 2 == 0 and N <= 8192)


def test_sliced_cases_reach_every_tile_of_slices(math):
    reached = set()
    for (D, _, _, F), (B, _, _, k) in [(d, r) for d in SLICED_DIMS for r in SLICED_ROWS] + [SLICED_ALONE]:
        reached |= {_slices(math, B * k, D, D, LAYERNORM)[1:], _slices(math, B * k, D, F, EITHER)[1:]}
    assert {cfg for cfg, splits in reached if splits > 1} == {16, 17, 34, 35, 40} and {splits for _, splits in reached} == {1, 2, 4, 8}


def test_attention_workgroups(math):
    """Up to 32 queries workgroups of 32 have half the waves that load keys and no more workgroups: over 257 to 1200 keys the launch
    was 1 to 6 % slower than on workgroups of 64."""
    for H in (16, 18, 32):
        for k in (1, 9, 31, 32):
            for L in (65, 128, 300, 600, 1200, 1536):
                assert math.attention(1, H, 128, k, L) == 3, (H, k, L)
            assert math.attention(1, H, 128, k, 1537) == 7 and math.attention(1, H, 128, k, 64) == 2
        assert math.attention(1, H, 128, 33, 300) == 7
    # both sides of the other lines
    for shape, cfg in [((1, 16, 128, 352, 521), 7), ((1, 16, 128, 353, 521), 3), ((4, 16, 128, 256, 512), 3), ((4, 16, 128, 256, 513), 5), ((3, 48, 128, 14, 575), 3), ((1, 18, 128, 222, 1103), 3),
                       ((1, 18, 128, 256, 1103), 7), ((1, 18, 128, 64, 1103), 7),
                       ((4, 16, 128, 257, 512), 5), ((4, 32, 128, 128, 513), 5), ((4, 32, 128, 128, 512), 3), ((1, 16, 64, 1024, 2624), 3),
                       ((1, 16, 64, 1025, 2624), 4), ((8, 30, 64, 410, 1626), 6), ((8, 30, 64, 300, 1626), 2), ((1, 64, 128, 4096, 9000), 6)]:
        assert math.attention(*shape) == cfg, (shape, cfg)


def test_attention_slices_of_head_dim_64(math):
    for shape, want in [((1, 16, 256, 641), 324), ((1, 16, 256, 640), 642), ((1, 16, 257, 897), 644), ((1, 16, 257, 896), 642), ((1, 16, 1024, 2624), 644),
                        ((4, 16, 257, 2624), 642), ((1, 30, 128, 700), 324), ((1, 30, 200, 700), 642), ((1, 30, 100, 1000), 324),
                        ((1, 30, 320, 2048), 642), ((1, 30, 320, 2049), 644), ((3, 7, 130, 1500), 324), ((1, 1, 1, 641), 324)]:
        assert math.attention_slices(*shape) == want, (shape, want)


def test_rows_of_a_restoring_wave(math):
    """A wave a row was 5 to 13 % slower than an unrolled pair for maps of many narrow rows, or of a width that deals the
    lines of a map to different XCDs."""
    for h, w, D in [(81, 82, 448), (97, 97, 448), (133, 155, 448), (66, 70, 64), (100, 104, 1024), (84, 88, 2048), (112, 120, 1536),
                    (72, 80, 1024)]:
        assert math.restore_rows(C.c_long(h * w), w, D) == -2, (h, w, D)
    for h, w, D in [(1, 1, 64), (16, 16, 1024), (53, 37, 2048), (64, 64, 2048), (65, 66, 448), (80, 80, 2048), (88, 96, 1280), (70, 93, 4096), (91, 95, 2048),
                    (104, 65, 2048)]:
        assert math.restore_rows(C.c_long(h * w), w, D) == 1, (h, w, D)
    for rows, w, D in [(128 * 128, 128, 2048), (90000, 300, 1920), (1 << 22, 2048, 8)]:
        assert math.restore_rows(C.c_long(rows), w, D) == 2, (rows, w, D)


@pytest.mark.parametrize("n", list(range(1, 20)) + list(range(60, 75)) + [1000, 4097, 8192])
def test_shares_of_the_xcds(math, n):
    """Every share is taken once, in runs by workgroups of one XCD for a contiguous run of them; what is left over is past the end.  Over eight
    samples every XCD has the same number of shares: the short run was always the same XCD's, and the others were waited for."""
    assert [math.xcd_share(i, n, 0, 3) for i in range(math.xcd_blocks(n, 0))] == list(range(n))
    assert not math.in_runs(n, 50, 1) if n < 64 else math.in_runs(n, 50, 1)
    blocks = math.xcd_blocks(n, 1)
    assert blocks % 8 == 0 and n <= blocks < n + 8
    taken = [0] * 8
    for sample in range(8):
        share = [math.xcd_share(i, n, 1, sample) for i in range(blocks)]
        assert sorted(share) == list(range(blocks))
        for xcd in range(8):
            first = share[xcd]
            assert share[xcd::8] == list(range(first, first + blocks // 8))
            taken[xcd] += sum(s < n for s in share[xcd::8])
    assert taken == [n] * 8


@pytest.mark.parametrize("rows", [1, 2])
def test_shares_in_turn_where_columns_meet_on_an_xcd(math, rows):
    """Shares dealt in turn are kept where most positions have the one below on their own XCD: widths near a multiple of 32 tokens a row of a
    wave.  At 48, 80 and 112 columns a wave of one row has it four XCDs away."""
    for w in range(1, 400):
        same = sum(n // (4 * rows) % 8 == (n + w) // (4 * rows) % 8 for n in range(32 * rows)) / (32 * rows)
        below = w > 16 * rows and same > 0.5   # (narrower: the next position is in the same share)
        assert math.in_runs(1000, w, rows) == (not below), (w, same)


def test_column_chunks_fit_the_scratch(math):
    """The sums of the chunks go to the head of an area for 32-row chunks, at most 256 of them."""
    for N in list(range(1, 700)) + [1024, 2047, 2048, 4095, 4096, 8192, 16384, 32767, 32768]:
        for D in (8, 64, 512, 1024, 1920, 2048, 4096, 8192):
            chunks = math.column_chunks(N, D)
            rows = -(-N // chunks)
            assert chunks in (1, 2, 4, 8, 16) and (chunks == 1 or rows >= 256)
            rows = 32 * -(-rows // 32)
            room = 32
            while -(-N // room) > 256:
                room *= 2
            assert -(-N // rows) <= -(-N // room), (N, D)


def test_attention_fetches_only_what_the_call_reads_later(math):
    """An attention half on its own, or a sub-layer step that keeps nothing in its MLP half, once fetched FC1's and FC2's weights too,
    past the end of whatever stood there for them."""
    out = (C.c_long * 4)()
    for D, F in [(64, 64), (1024, 4096), (1920, 7680), (2048, 8192), (2304, 6912), (4096, 16384)]:
        for M in (1, 16, 17, 130, 576, 4096):
            for in_stack in (0, 1):
                math.ahead(D, F, M, in_stack, 0, out)
                assert out[0] <= 1 and (out[0] == 0 or out[1] == 2 * D * D), (D, F, M, in_stack)
                math.ahead(D, F, M, in_stack, 1, out)
                large = 2 * D * F >= 16 << 20
                assert out[0] == (3 if large or (in_stack and M > 16) else 0)
                assert out[0] == 0 or tuple(out)[1:] == (2 * D * D, 2 * D * F, 2 * D * F)


@pytest.mark.parametrize("cut", [0, 1])
def test_prefetch_plan_stays_inside_the_list_and_the_idle_units(math, cut):
    """Whole matrices in their order (or, cut, a prefix of the bytes), never more workgroups than idle units, none for nothing."""
    out = (C.c_long * 2)()
    for sizes in ([], [0], [100], [8 << 20, 32 << 20, 32 << 20], [2 << 20, 8 << 20, 8 << 20], [1 << 40], [0, 0, 64], [127, 1 << 20]):
        prefixes = {sum(sizes[:i]) for i in range(len(sizes) + 1)}
        for idle in (-5, 0, 1, 7, 8, 64, 76, 192, 255):
            for us in (0.0, 6.5, 7.95, 23.9, 1000.0):
                math.prefetch((C.c_long * max(1, len(sizes)))(*sizes), len(sizes), idle, C.c_double(us), cut, out)
                got, blocks = out
                assert 0 <= got <= sum(sizes) and 0 <= blocks <= max(0, idle) and (got > 0) >= (blocks > 0)
                assert blocks > 0 or got == 0
                assert cut or got in prefixes, (sizes, idle, us, got)
