"""csrc/split.h, compiled for the host: how work is divided between workgroups."""
from __future__ import annotations

import ctypes as C
import os
import subprocess

import pytest

from paper_2406_06220_amd import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include "split.h"
using namespace tdt;
extern "C" void pred_share_c(int deep, int nt_a, int nt_b, int h_pred, int C, int rank, int *out)
{
    const PredShare s = pred_share(deep != 0, nt_a, nt_b, h_pred, C, rank);
    const int v[6] = {s.qt0, s.na, s.r0, s.nr, s.u0, s.U};
    for (int i = 0; i < 6; ++i) out[i] = v[i];
}
extern "C" void group_split_c(int general, int bf16, int lstm, int layers, int h_joint, int h_pred, int outputs, int B,
                              int streaming_least, int frame_loop, int on_the_fly, int window, int joint_tiles, int *out)
{
    const SplitModel m = split_model(bf16 != 0, lstm != 0, layers, h_joint, h_pred, outputs);
    const GroupSplit s = general ? general_split(m, B, 256, streaming_least, frame_loop != 0, on_the_fly != 0)
                                 : label_split(m, B, 256, streaming_least, JointAsked{window, joint_tiles});
    const int v[3] = {s.n_clusters, s.one_workgroup, s.window_most};
    for (int i = 0; i < 3; ++i) out[i] = v[i];
}
extern "C" int window_c(int general, int C, int nt, int hyps, int hpc, int n, int window, int rows_cap, int most)
{
    return general ? general_window(n, window, general_joint_rows(general == 1, C, nt, 0, hyps), rows_cap, most)
                   : label_window(n, window, label_joint_rows(C, nt, 0, hpc), rows_cap, C, nt);
}
extern "C" void nowhere_c(int *out)
{
    const int v[3] = {kNowhere, kLabelLongest, label_nk(true, kLabelLongest) > 0 && label_nk(true, kLabelLongest + 1) == 0};
    for (int i = 0; i < 3; ++i) out[i] = v[i];
}
extern "C" int few_rows_c(bool bf16, int k, int per_wg, int hpc, int h_pred) { return few_rows(label_nk(bf16, k), per_wg, hpc, h_pred); }
extern "C" int wide_round_c(int layers, int nt_a, int nt_b, int C) { return wide_round(layers, nt_a, nt_b, C) ? kWideRound : 0; }
extern "C" long long planes_covered_c(int n_clusters, int h_pred, int hpc, int nk) { return planes_covered(n_clusters, h_pred, hpc, nk); }
extern "C" void planes_c(int h_pred, int hpc, int steps, int s, int *out)
{
    const int v[3] = {plane_step(hpc), plane_bytes(h_pred, hpc), plane_step_at(plane_step(hpc), steps, s)};
    for (int i = 0; i < 3; ++i) out[i] = v[i];
}
extern "C" void words_c(int wide, int durations, int n_clusters, int hpc, int C, long long *out)
{
    const LabelWords w = label_words(wide != 0, durations != 0, n_clusters, hpc, C);
    const long long v[7] = {w.rows, w.cells, w.lse, w.dur, w.present, w.end, kLabelWordsMost};
    for (int i = 0; i < 7; ++i) out[i] = v[i];
}
extern "C" int in_order_c(int launch, long long row_tiles, long long column_tiles)
{
    return tiles_in_order(launch == 0 ? TileLaunch::kPrepare : launch == 1 ? TileLaunch::kOwn : TileLaunch::kSmall, row_tiles,
                          column_tiles);
}
extern "C" int big_tiles_c(int ragged, long long rows, long long column_tiles) { return big_tiles(ragged != 0, rows, column_tiles); }
extern "C" int long_window_c() { return kLongWindow; }
extern "C" int item_c(int C, int nt, int hpc, int window, int joint_tiles)
{
    return usual_item(C, nt, hpc, window, joint_tiles, hpc * 64 < 256 ? hpc * 64 : 256);
}
"""


@pytest.fixture(scope="module")
def split(tmp_path_factory):
    d = tmp_path_factory.mktemp("split")
    src, lib = str(d / "split.cpp"), str(d / "libsplit.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-Wall", "-Werror",
                    "-I", os.path.join(ROOT, "paper_2406_06220_amd", "csrc"), src, "-o", lib], check=True)
    return C.CDLL(lib)


@pytest.mark.parametrize("deep", [0, 1])
@pytest.mark.parametrize("H,Hp", [(8, 8), (16, 40), (48, 40), (640, 640), (24, 1024), (1024, 8), (264, 200)])
def test_predictor_side_is_dealt_out_whole(split, deep, H, Hp):
    """Every column tile and hidden unit has one owner, and no workgroup points at a unit the model does
    not have: all of them request the per-label table from their first unit on."""
    nt_a, nt_b = -(-H // 16), -(-Hp // 4)
    out = (C.c_int * 6)()
    for n in (1, 2, 3, 7, 16, 51, 85, 128, 255, 256):
        tiles_a, tiles_b, units = [], [], []
        for rank in range(n):
            split.pred_share_c(deep, nt_a, nt_b, Hp, n, rank, out)
            qt0, na, r0, nr, u0, U = out
            assert na >= 0 and nr >= 0 and U >= 0
            tiles_a += range(qt0, qt0 + na)
            tiles_b += range(r0, r0 + nr)
            units += range(u0, u0 + U)
            assert 0 <= u0 and u0 + max(U, 1) <= Hp, (n, rank)
        assert tiles_a == list(range(nt_a)) and tiles_b == list(range(nt_b)) and units == list(range(Hp))


def test_stateless_predictor_has_no_share(split):
    out = (C.c_int * 6)()
    split.pred_share_c(0, 40, 0, 640, 9, 4, out)
    assert list(out) == [0] * 6


def group_split(split, cfg, general=0, on_the_fly=0, streaming=0, frame_loop=0, window=0, joint_tiles=0):
    out = (C.c_int * 3)()
    split.group_split_c(general, int(cfg.dtype == "bf16"), int(cfg.pred_kind == "lstm"), cfg.pred_layers, cfg.h_joint, cfg.h_pred,
                        cfg.n_out, cfg.B, 4 * streaming, frame_loop, on_the_fly, window, joint_tiles, out)
    return list(out)


def test_group_counts_of_the_benchmark_models(split):
    got = [group_split(split, c) for c in (synth.CFG1, synth.CFG2, synth.CFG3, synth.CFG4, synth.CFG2_B128,
                                           synth.CFG2.with_batch(1), synth.CFG2.with_batch(7), synth.CFG2.with_batch(256))]
    assert got == [[4, 1, 64], [5, 0, 64], [5, 0, 64], [28, 0, 64], [8, 0, 64], [2, 0, 64], [5, 0, 64], [16, 0, 64]]
    assert group_split(split, synth.CFG5, streaming=1) == [16, 0, 64]


@pytest.mark.parametrize("general", [0, 1])
@pytest.mark.parametrize("kind", ["lstm", "stateless"])
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_group_counts_over_all_sizes(split, kind, general, dtype):
    """Groups exist, hold what they may hold, and the general kernel's are never single workgroups: with
    all of the chip's workgroups dealt out, a group of it has more than one while it can."""
    for vocab in (1, 40, 63, 64, 1024, 9000):
        for H, Hp in ((8, 8), (640, 640), (2048, 1024)):
            for B in (1, 2, 3, 15, 16, 64, 111, 112, 300, 1500, 16640, 65536):
                for streaming, frame_loop in ((0, 0), (1, 0), (0, general)):
                    cfg = synth.small_config("split", dtype=dtype, pred_kind=kind, vocab=vocab, h_joint=H, h_pred=Hp, emb_dim=Hp, B=B)
                    n, one, most = group_split(split, cfg, general, 0, streaming, frame_loop)
                    assert 1 <= n <= 256 and -(-B // n) <= 256 and most == 64
                    assert not (general and one) and (not one or n == min(B, 256))
                    if general and B <= 64 * 64:
                        assert 256 // n >= 2


def test_projections_on_the_fly_of_small_output_layers(split):
    """One hypothesis a group and one row tile a pass, as its group of one workgroup has by default."""
    for B in (4, 60):
        cfg = synth.CFG1.with_batch(B)
        assert group_split(split, cfg) == [B, 1, 64]
        assert group_split(split, cfg, general=1, on_the_fly=1) == [B, 0, 16]


def test_group_counts_of_the_general_kernel(split):
    """Where its rules leave the label loop's."""
    b256 = synth.CFG2.with_batch(256)
    assert group_split(split, b256)[0] == 16 and group_split(split, b256, general=1)[0] == 8
    assert group_split(split, b256, general=1, frame_loop=1)[0] == 16
    assert [group_split(split, synth.CFG4.with_batch(32), general=1, frame_loop=f)[0] for f in (0, 1)] == [11, 23]
    assert group_split(split, synth.CFG1.with_batch(32), general=1)[0] == 16


def test_windows(split):
    """A window has at least a frame, at most 64 or the longest asked for, keeps its pass within the row limit and
    fills the row tiles it needs; the general kernel's items take eight column tiles (config 2: 11 frames
    of seven hypotheses), the label loop's four there (six frames)."""
    assert split.window_c(1, 51, 65, 7, 7, 7, 0, 448, 64) == 11 and split.window_c(0, 51, 65, 7, 7, 7, 0, 256, 64) == 6
    assert split.window_c(2, 51, 65, 7, 7, 7, 0, 448, 64) == 6   # (float32: four tiles)
    for general, cap in ((1, 1024), (2, 1024), (0, 256)):
        for C_ in (1, 2, 9, 17, 51, 128, 256):
            for nt in (1, 4, 5, 65, 513):
                for hyps in (1, 4, 5, 16, 64):
                    rows_cap = min(hyps * 64, cap)
                    for n in range(1, hyps + 1):
                        for window, most in ((0, 64), (0, 16), (1, 64), (64, 64)):
                            w = split.window_c(general, C_, nt, hyps, hyps, n, window, rows_cap, most)
                            assert 1 <= w <= 64 and w * n <= rows_cap
                            if window:
                                assert w == min(window, rows_cap // n)
                            elif general:
                                assert w <= most
                            if not window and w < (most if general else 64) and w * n <= rows_cap - n:
                                assert -(-n * (w + 1) // 16) > -(-n * w // 16)   # (a frame more takes a row tile more)


def test_an_offset_that_is_nowhere(split):
    """It lies beyond the largest exchange buffer and stays a positive number with any offset inside a row added."""
    out = (C.c_int * 3)()
    split.nowhere_c(out)
    nowhere, longest, longest_taken = out
    assert longest_taken
    assert nowhere + 4 * longest < 2 ** 31
    assert nowhere >= 2 * 4 * 256 * 64 * longest * 4


def test_usual_items(split):
    """65 column tiles.  One frame a pass: 32 of 64 hypotheses are two row tiles, a workgroup each of 128 for a column
    tile and one over; by default items of the tiles the window aims at, and never more than there are."""
    assert [split.item_c(C_, 65, hpc, 1, 0) for C_, hpc in ((256, 32), (128, 64), (85, 43), (51, 26), (32, 16), (16, 8))] == [1, 2, 2, 2, 3, 5]
    assert [split.item_c(C_, 65, hpc, 0, 0) for C_, hpc in ((51, 5), (9, 5), (9, 2), (256, 1))] == [4, 8, 8, 2]
    for C_ in (1, 2, 9, 51, 256):
        for nt in (5, 65, 255):
            for hpc in (1, 2, 16, 63, 64):
                for window in (0, 1, 8, 64):
                    assert -(-nt // C_) <= split.item_c(C_, nt, hpc, window, 0) <= nt


@pytest.mark.parametrize("hpc", [1, 4, 5, 8, 9, 16])
def test_no_step_of_the_hidden_state_lies_beyond_its_buffer(split, hpc):
    """The scalar offset of every load of the hidden state's terms, over all widths, of steps that a wavefront has and of those
    that are only compiled: never past the buffer's end, which the last buffer shares with the descriptor; and the steps that
    wavefronts have are all there are, each once."""
    out = (C.c_int * 3)()
    for h_pred in range(8, 1025, 8):
        steps = -(-h_pred // 32)
        for nk in (5, 8):
            if steps > 4 * nk:
                continue
            seen = []
            for wave in range(4):
                have = steps // 4 + (wave < steps % 4)
                first = wave * (steps // 4) + min(wave, steps % 4)
                for s in range(nk):
                    split.planes_c(h_pred, hpc, have, s, out)
                    step, size, at = out[0], out[1], first * out[0] + out[2]
                    assert 0 <= at <= size, (h_pred, nk, wave, s)
                    if s < have:
                        seen.append(at)
            assert seen == [i * step for i in range(steps)] and size == steps * step


@pytest.mark.parametrize("hpc", [1, 4, 5, 8, 9, 16])
def test_what_the_descriptor_of_the_terms_covers(split, hpc):
    """Reductions over 640 leave the scalar offset of a compiled step that a wavefront does not have where it falls: always before the end
    of what the descriptor covers, in the last group's second buffer as well.  Up to 640 it covers the buffers and nothing else."""
    split.planes_covered_c.restype = C.c_longlong
    out = (C.c_int * 3)()
    for h_pred in range(8, 1025, 8):
        steps, n = -(-h_pred // 32), 64 // hpc
        split.planes_c(h_pred, hpc, steps, 0, out)
        step, size = out[0], out[1]
        covered = split.planes_covered_c(n, h_pred, hpc, 8)
        for wave in range(4):
            first = wave * (steps // 4) + min(wave, steps % 4)
            assert (2 * n - 1) * size + (first + 7) * step < covered <= 2 * n * size + 8 * step
        assert split.planes_covered_c(n, h_pred, hpc, 5) == 2 * n * size


def test_rows_that_are_multiplied_four_at_a_time(split):
    """float32, one LSTM layer: up to eight rows with the longer reductions; with the shorter ones, whose products of sixteen rows
    are soon done, up to four, where they take more than half a round of column tiles and three steps or four a wavefront."""
    for k, hp in ((264, 264), (264, 8), (640, 128), (640, 640)):
        assert [split.few_rows_c(0, k, per, hpc, hp) for per in (1, 4) for hpc in (1, 4, 5, 8, 9, 16)] == [1, 1, 1, 1, 0, 0] * 2
    for k, hp in ((136, 129), (256, 136), (256, 256)):
        assert [[split.few_rows_c(0, k, per, hpc, hp) for hpc in (1, 4, 5, 8, 9)] for per in (1, 2, 3, 4, 5, 8)] == [[0] * 5] * 2 + [[1, 1, 0, 0, 0]] * 4
    for k, hp in ((8, 8), (120, 120), (256, 128), (256, 64)):
        assert not any(split.few_rows_c(0, k, per, hpc, hp) for hpc in (1, 4, 8) for per in (1, 3, 4, 8))


def test_one_round_of_eight_wavefronts(split):
    """Where a workgroup's column tiles are said to be one round, no workgroup has more; with as many groups as batches of one
    layer get by themselves that is four groups of 640 or of 1024 units, and not more of them."""
    out = (C.c_int * 6)()
    rounds = 0
    for H in range(8, 1025, 72):
        for Hp in range(8, 1025, 56):
            for n in (1, 2, 7, 16, 32, 64, 128, 256):
                nt_a, nt_b = -(-H // 16), -(-Hp // 4)
                most = split.wide_round_c(1, nt_a, nt_b, n)
                assert not split.wide_round_c(2, nt_a, nt_b, n)
                rounds += most > 0
                for rank in range(n if most else 0):
                    split.pred_share_c(1, nt_a, nt_b, Hp, n, rank, out)
                    assert out[1] + out[3] <= most, (H, Hp, n, rank)
    assert rounds > 100
    assert [split.wide_round_c(1, 40, 160, n) > 0 for n in (128, 64, 32, 16)] == [True, True, False, False]
    assert [split.wide_round_c(1, 64, 256, n) > 0 for n in (128, 64, 32, 16)] == [True, True, False, False]


def label_groups(split, B, dtype="bf16", kind="lstm", layers=1, H=640, Hp=640, n_out=1025, **asked):
    cfg = synth.small_config("split", dtype=dtype, pred_kind=kind, pred_layers=layers, h_joint=H, h_pred=Hp, emb_dim=Hp, vocab=n_out - 1, B=B)
    n, one, _ = group_split(split, cfg, **asked)
    assert not one
    return n


def test_group_counts_of_one_lstm_layer(split):
    """Where five groups fit: five already in small batches while a group's workgroups have at most two rounds of column
    tiles; three hypotheses in three groups where that makes no second round of one; never more groups than
    hypotheses but for one alone.  Two layers, widths that leave a workgroup more tiles (and with them not the
    one-layer form), models that more groups fit: four at most."""
    groups = lambda B, **kw: label_groups(split, B, **kw)
    batches = (1, 2, 3, 4, 5, 7, 15, 16, 32, 128)
    one_round, two_rounds, four = [2, 2, 3, 4, 5, 5, 5, 5, 5, 8], [2, 2, 2, 4, 5, 5, 5, 5, 5, 8], [2, 2, 2, 4, 4, 4, 4, 5, 5, 8]
    for H, Hp in ((640, 640), (448, 640), (640, 592)):
        assert [groups(B, H=H, Hp=Hp) for B in batches] == one_round, (H, Hp)
        assert [groups(B, H=H, Hp=Hp, dtype="fp32") for B in batches] == two_rounds, (H, Hp)
    for H, Hp in ((648, 648), (1024, 512), (128, 768)):
        assert [groups(B, H=H, Hp=Hp) for B in batches] == two_rounds, (H, Hp)
    for H, Hp in ((704, 704), (1024, 640), (512, 768)):
        assert [groups(B, H=H, Hp=Hp) for B in batches] == four, (H, Hp)
    assert [groups(B, layers=2) for B in batches] == four
    assert [groups(B, H=48, Hp=40) for B in (1, 3, 5, 15)] == [2, 2, 4, 4]   # (many would fit)
    assert [groups(B, H=768, Hp=768) for B in (2, 3, 4, 5, 15, 16)] == [2, 2, 4, 4, 4, 4]
    assert [groups(B, H=1024, Hp=1024) for B in (2, 3, 4, 5, 15, 16)] == [2, 3, 3, 3, 3, 3]


def test_group_counts_by_the_joint_passes(split):
    """One LSTM layer of 640: four groups where the windows of five would hold fewer row tiles, or a caller's window
    would make their items take more rounds; windows of more than eight frames by the general rule."""
    groups = lambda B, n_out, window=0, joint_tiles=0, **kw: label_groups(split, B, n_out=n_out, window=window, joint_tiles=joint_tiles, **kw)
    for dtype in ("bf16", "fp32"):
        assert [groups(9, n_out, dtype=dtype) for n_out in (128, 501, 1025, 1088, 2001, 3300, 4091)] == [5, 4, 5, 5, 4, 4, 4]
        assert [groups(15, n_out, dtype=dtype) for n_out in (128, 501, 1025, 2001, 4091)] == [5, 4, 5, 4, 5]
    assert [groups(9, 1025, window=w) for w in (1, 4, 8, 9, 64)] == [5, 5, 5, 4, 4]
    assert [groups(9, 4091, window=w) for w in (1, 4, 8, 9, 64)] == [4, 4, 4, 4, 4]
    assert [groups(3, 1025, window=w) for w in (0, 1, 8, 9, 64)] == [3, 3, 3, 2, 2]
    assert [groups(9, 501, joint_tiles=j) for j in (1, 4, 8)] == [4, 4, 5]


def test_group_counts_of_stateless_models(split):
    """Eight column tiles a round: few groups with items of four tiles on three row tiles while that leaves five
    hypotheses a group and gives five to twenty of them, then groups by items of eight and twelve tiles.  A caller's
    window of up to eight frames or size of the items: the groups of the other stateless forms instead of the few."""
    groups = lambda B, n_out=1025, **kw: label_groups(split, B, kind="stateless", n_out=n_out, **kw)
    assert [groups(B) for B in (1, 4, 25, 26, 32, 140, 141, 256)] == [5, 4, 5, 26, 28, 28, 42, 42]
    assert [groups(B, n_out=501) for B in (16, 48, 50, 51, 128)] == [10, 10, 10, 51, 64]
    assert [groups(B, n_out=128) for B in (16, 48, 128)] == [16, 48, 64]
    assert [groups(B, n_out=2049) for B in (4, 8, 10, 11, 24)] == [3, 3, 5, 11, 15]
    assert [groups(24, window=w) for w in (0, 1, 8, 9, 64)] == [5, 11, 11, 5, 5]
    assert [groups(24, joint_tiles=j) for j in (0, 1, 8)] == [5, 11, 11]
    assert [groups(64, window=w) for w in (0, 1, 64)] == [28, 28, 28]
    assert [groups(24, dtype="fp32", window=w) for w in (0, 1, 64)] == [11, 11, 11]
    for n_out in (80, 128, 256, 1024, 1025, 3200, 16400):
        for B in (*range(1, 70), 128, 500, 20000):
            for kind in ("lstm", "stateless"):
                for asked in ({}, dict(window=1), dict(window=64), dict(joint_tiles=1)):
                    n = label_groups(split, B, kind=kind, n_out=n_out, **asked)
                    assert max(1, -(-B // 256)) <= n <= max(64, -(-B // 256)) and (n <= B or B == 1), (kind, n_out, B, asked)


def test_words_of_the_joint_passes_are_reached_by_32_bit_offsets(split):
    """Arrays that do not overlap and hold every word, and no split of the chip's workgroups has more than the bound."""
    out, most = (C.c_longlong * 7)(), 0
    for n in range(1, 257):
        for c in sorted({1, 2, 3, 15, 16, 17, 64, 128, 255, 256, 256 // n}):
            if n * c > 256:
                continue
            for hpc in (1, 3, 4, 16, 64, 256):
                for wide in (0, 1):
                    for dur in (0, 1):
                        split.words_c(wide, dur, n, hpc, c, out)
                        rows, cells, lse, durs, present, end, bound = out
                        assert rows == min(64 * hpc, 256) and cells >= max(rows, 16 * c) and cells % 16 == 0
                        assert lse >= n * 4 * cells * 8 and durs >= lse + n * 4 * cells * 8
                        assert present >= durs + dur * n * 4 * 2 * rows * 8 and end >= present + n * 5 * c * 8
                        assert all(x % 256 == 0 for x in (lse, durs, present, end)) and end <= bound
                        most = max(most, end)
    assert most > 0.99 * bound and bound < 2**31 - 2**16


def test_order_of_a_projections_tiles(split):
    """Row tiles are given out in order only where it was measured to pay: in the preparation launch, and elsewhere where
    dealing them fills a die's compute units before the others'; never from 24 row tiles on."""
    order = lambda launch, r, c: split.in_order_c(launch, C.c_longlong(r), C.c_longlong(c)) != 0   # noqa: E731
    prepare, own, small = 0, 1, 2
    for r in range(1, 40):
        for c in (1, 5, 20, 40):
            assert order(prepare, r, c) == (r < 24)
    for r, c in ((1, 4), (2, 10), (1, 16), (6, 16), (12, 16), (21, 16), (23, 16), (1, 32), (8, 32), (16, 32)):
        assert order(own, r, c)
    for r, c in ((21, 8), (23, 8), (3, 10), (17, 10), (23, 10), (23, 4), (24, 16), (32, 32)):
        assert not order(own, r, c)
    for r, c in ((1, 2), (1, 10), (1, 16), (2, 16), (1, 20), (2, 20), (2, 32), (9, 20), (12, 20)):
        assert order(small, r, c)
    for r, c in ((6, 10), (8, 10), (9, 10), (16, 10), (20, 10), (23, 10), (28, 10), (3, 16), (8, 16), (16, 16), (23, 16), (23, 2), (9, 4), (23, 4),
                 (6, 8), (16, 8), (23, 8), (3, 20), (8, 20), (13, 20), (16, 20), (23, 20), (8, 32), (16, 32)):
        assert not order(small, r, c)


def test_large_tiles_where_neither_full_nor_half_padded_batches_lose(split):
    """129 tiles of valid rows are where 256 x 256 tiles begin to pay.  Batches whose lengths nobody knows on the host take
    them where lengths even over a tenth to the whole fill as many."""
    big = lambda ragged, rows, c: split.big_tiles_c(ragged, C.c_longlong(rows), C.c_longlong(c)) != 0   # noqa: E731
    for c in (2, 3, 4, 5, 8):
        for tiles in range(100, 400):
            rows = tiles * 256 // c
            if rows < 32768:
                assert big(0, rows, c) == (-(-rows // 256) * c >= 160)
                if big(1, rows, c):
                    assert 0.55 * rows / 256 * c > 129
                elif -(-rows // 256) * c >= 260:
                    raise AssertionError((rows, c))
            else:
                assert big(0, rows, c) and big(1, rows, c)
    assert big(1, 32768, 1) and not big(1, 32767, 1) and not big(0, 32512, 1)


def test_a_hypothesis_of_its_own_has_a_long_window(split):
    """Whether hypotheses go on before all of their group have found a label is decided by the window that all of them would
    search with.  One alone never does: it has nobody to wait for."""
    for C_ in (1, 2, 3, 7, 15, 16, 17, 32, 51, 64, 128, 256):
        for nt in (1, 4, 5, 9, 33, 65, 129, 513, 2048):
            for hpc in (1, 2, 5, 16, 64):
                assert split.window_c(0, C_, nt, hpc, hpc, 1, 0, min(64 * hpc, 256), 64) >= split.long_window_c()
