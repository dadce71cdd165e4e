"""The label-looping kernel of csrc/label_loop.hip where its forms meet: groups that fill or just
exceed what one staging tile packs or holds, reductions at the borders of its compiled lengths,
output layers at the borders of a round of column tiles, groups of one workgroup, passes of more rows
than a wavefront has lanes, and what falls back to the general kernel -- against the oracle."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2406_06220_amd import synth
from test_gpu_parity import check, gpu, run_gpu  # noqa: F401  (gpu: the fixture)

pytestmark = pytest.mark.gpu


def config(name, **kw):
    base = dict(dtype="bf16", pred_kind="lstm", d_enc=32, h_pred=40, emb_dim=24, h_joint=48, vocab=70, B=12, T=30,
                len_lo=0, len_hi=30, seed=300, default_blank_bias=1.0, max_symbols=4)
    base.update(kw)
    return synth.small_config(name, **base)


CASES = [
    # hypotheses of one group: packed planes up to 4, one row per wavefront pair up to 8, one row tile up
    # to 16, several row tiles, the most a lane holds, and beyond it
    *[(config(f"ll_group{n}", B=n), dict(n_clusters=1)) for n in (1, 4, 5, 8, 9, 16, 17, 33, 64, 65)],
    # more than one cell a thread; more column tiles a workgroup than a round
    (config("ll_cells", h_pred=320, B=30), dict(n_clusters=15)),
    (config("ll_rounds", h_pred=320, B=60), dict(n_clusters=60)),
    # groups of one and of two workgroups
    (config("ll_c1", B=256, T=8, len_hi=8), dict(n_clusters=256)),
    (config("ll_c1_tdt", B=250, T=9, len_hi=9, durations=(0, 1, 2)), dict(n_clusters=250)),
    (config("ll_c2", B=128, T=8, len_hi=8, durations=(0, 1, 3)), dict(n_clusters=128)),
    # reductions: one step, the compiled lengths and one input group beyond, the longest
    *[(config(f"ll_k{h}_{hp}", h_joint=h, h_pred=hp, emb_dim=24, B=5), {})
      for h, hp in ((8, 8), (32, 648), (640, 640), (648, 32), (1024, 1000), (1032, 40))],
    # column tiles: a multiple, one column more, duration outputs across a tile border
    *[(config(f"ll_v{v}_{len(d)}", vocab=v, durations=d, B=7), dict(n_clusters=c))
      for v, d, c in ((63, (), 7), (64, (), 7), (254, (0, 1, 2), 7), (1021, (0, 1, 2, 3, 4), 2))],
    # passes of more than 64 rows, windows cut by the row limit
    (config("ll_rows", B=30, durations=(1, 2)), dict(n_clusters=2, window=8)),
    (config("ll_rows_cap", B=50), dict(n_clusters=1, window=64)),
    # stateless predictors, one and two labels of context
    (config("ll_stateless1", pred_kind="stateless", pred_layers=1, h_pred=24, B=20), {}),
    # score terms still being summed while the next pass is exchanged: many hypotheses a workgroup, one workgroup
    (config("ll_stateless_many", pred_kind="stateless", pred_layers=1, h_pred=24, B=2100, T=14, len_hi=14), {}),
    (config("ll_stateless_c1", pred_kind="stateless", pred_layers=1, h_pred=24, B=256, T=20, len_hi=20),
     dict(n_clusters=256, window=2)),
    (config("ll_stateless2", pred_kind="stateless", pred_layers=2, h_pred=48, B=70, durations=(0, 2)), {}),
    (config("ll_mb_stateless", pred_kind="stateless", pred_layers=2, h_pred=48, B=9, durations=(2, 4), multi_blank=True),
     dict(n_clusters=1)),
    # float32: the compiled lengths and one input group beyond, several rounds of column tiles, row tiles
    *[(config(f"ll_f32_k{h}_{hp}", dtype="fp32", h_joint=h, h_pred=hp, B=5), {})
      for h, hp in ((8, 8), (256, 72), (264, 248), (640, 640), (648, 32))],
    # float32: wavefronts with fewer steps than are compiled, with none, and not all with the same number
    *[(config(f"ll_f32_steps{h}_{hp}", dtype="fp32", h_joint=h, h_pred=hp, B=9, vocab=150), dict(n_clusters=c))
      for h, hp, c in ((16, 64, 1), (80, 24, 2), (128, 200, 1), (192, 256, 9))],
    (config("ll_f32_rounds", dtype="fp32", h_pred=96, h_joint=272, vocab=260, durations=(0, 1, 2), B=40), dict(n_clusters=2)),
    (config("ll_f32_deep", dtype="fp32", pred_layers=2, B=20), dict(n_clusters=4)),
    # rows staged for the matrix cores: half a row tile of hypotheses and both halves, reductions that end inside a
    # 128-byte piece, one staging area and two; stateless: more than eight hypotheses in a row tile
    *[(config(f"ll_staged_k{h}_{hp}_{B}", h_joint=h, h_pred=hp, B=B), dict(n_clusters=1))
      for h, hp, B in ((8, 16, 16), (104, 616, 7), (616, 640, 13), (648, 40, 8), (1000, 1024, 16))],
    *[(config(f"ll_staged_f32_k{h}_{hp}_{B}", dtype="fp32", h_joint=h, h_pred=hp, B=B), dict(n_clusters=1))
      for h, hp, B in ((8, 8, 9), (248, 256, 16), (632, 280, 7), (264, 640, 12))],
    *[(config(f"ll_staged_{t}_stateless{n}_k{h}_w{w}", dtype=t, pred_kind="stateless", pred_layers=n, emb_dim=24, h_pred=24 * n,
              h_joint=h, vocab=200, B=20), dict(n_clusters=1, window=w))
      for t, n, h, w in (("bf16", 1, 616, 1), ("bf16", 2, 648, 1), ("bf16", 2, 1024, 2), ("fp32", 2, 248, 1), ("fp32", 1, 640, 3))],
    # weights that stay in registers: few searching hypotheses move the work items to other column tiles, items of one
    # round, two and three, phase Q of one and two rounds
    *[(config(f"ll_kept_{t}_v{v}_{B}_{c}", dtype=t, h_pred=hp, vocab=v, B=B, T=40, len_lo=1, len_hi=40), dict(n_clusters=c, joint_tiles=j))
      for t, hp, v, B, c, j in (("bf16", 320, 1000, 40, 5, 4), ("bf16", 320, 1000, 60, 10, 8), ("bf16", 320, 700, 32, 16, 12),
                                ("fp32", 320, 500, 40, 5, 4), ("fp32", 96, 900, 48, 16, 8))],
    # the same, one layer with two rounds of phase Q: joint items of one round to four, reductions of both lengths
    *[(config(f"ll_two_rounds_{t}_{h}_{hp}_v{v}_{B}_{c}", dtype=t, h_joint=h, h_pred=hp, vocab=v, B=B, T=20, len_lo=1, len_hi=20), dict(n_clusters=c, joint_tiles=j))
      for t, h, hp, v, B, c, j in (("bf16", 48, 320, 60, 40, 16, 1), ("bf16", 48, 320, 900, 208, 16, 15), ("bf16", 640, 640, 1000, 100, 8, 8),
                                   ("bf16", 648, 648, 500, 60, 4, 2), ("bf16", 648, 648, 1000, 60, 4, 8), ("bf16", 1000, 128, 300, 39, 4, 8),
                                   ("fp32", 48, 248, 900, 40, 16, 15), ("fp32", 272, 320, 500, 60, 10, 8), ("fp32", 640, 640, 300, 30, 5, 4))],
    *[(config(f"ll_kept_stateless_v{v}_{c}", pred_kind="stateless", h_pred=24, vocab=v, B=60, T=40, len_lo=1, len_hi=40),
       dict(n_clusters=c, joint_tiles=j)) for v, c, j in ((1000, 20, 8), (1000, 30, 12), (300, 60, 4))],
    # one staging area and the predictor's rows as they are fed: one to sixteen different ones in a row tile, reductions
    # that end inside a step, one round of phase Q and two
    *[(config(f"ll_fed_k{h}_{hp}_{B}_{c}_w{w}", h_joint=h, h_pred=hp, B=B, T=24, len_lo=1, len_hi=24), dict(n_clusters=c, window=w))
      for h, hp, B, c, w in ((648, 40, 1, 1, 64), (648, 40, 16, 1, 1), (1000, 1024, 15, 1, 3), (1024, 648, 8, 1, 0), (1016, 64, 9, 1, 2),
                             (648, 648, 44, 4, 1), (1024, 320, 20, 3, 5))],
    # planes with two rounds of phase Q: one to eight rows, a second round of one tile and of all
    *[(config(f"ll_planes2_k{h}_{hp}_{B}_{c}", h_joint=h, h_pred=hp, B=B, T=24, len_lo=1, len_hi=24), dict(n_clusters=c))
      for h, hp, B, c in ((48, 320, 16, 16), (48, 320, 48, 16), (48, 320, 64, 16), (48, 248, 80, 16), (16, 256, 112, 16), (48, 496, 128, 16),
                          (648, 648, 4, 4), (648, 648, 16, 4), (1024, 1000, 10, 2), (616, 704, 28, 4), (648, 696, 32, 4))],
    # stateless work items of one to four column tiles, of six and seven in passes of all hypotheses only, and at the border to
    # the form that takes eight at once; duration outputs in an item of their own
    *[(config(f"ll_items_stateless{n}_v{v}_{B}_{c}_w{w}", pred_kind="stateless", pred_layers=n, emb_dim=24, h_pred=24 * n, h_joint=h,
              vocab=v, durations=d, B=B, T=16, len_hi=16), dict(n_clusters=c, window=w))
      for n, h, v, d, B, c, w in ((1, 48, 1000, (), 10, 1, 1), (2, 640, 1021, (0, 1, 2, 3, 4), 40, 1, 2), (1, 72, 1000, (), 60, 1, 3),
                                  (2, 48, 1000, (1, 2), 60, 1, 4), (1, 616, 1000, (), 150, 3, 2), (2, 48, 1021, (0, 2), 160, 3, 2),
                                  (1, 48, 1000, (), 30, 1, 0), (2, 104, 300, (), 12, 4, 0))],
    # column groups at the borders of what a lane of the gather takes at a time: 16, 17, 24, 25, 49
    *[(config(f"ll_column_groups{n}", vocab=n * 16 - 2, B=6, T=20, len_hi=20), dict(n_clusters=1, joint_tiles=1, window=w))
      for n, w in ((16, 8), (17, 8), (24, 8), (25, 8), (49, 8), (40, 1))],
    # few rows of the hidden state, staged as planes: one to eight, reductions that end inside a step and that leave
    # wavefronts without one, one column tile and all of a round
    *[(config(f"ll_planes_k{h}_{hp}_{B}", h_joint=h, h_pred=hp, B=B), dict(n_clusters=c))
      for h, hp, B, c in ((8, 8, 1, 1), (40, 616, 3, 1), (640, 632, 4, 1), (104, 640, 5, 1), (616, 24, 7, 1), (640, 640, 8, 1),
                          (1024, 1000, 8, 1), (648, 1024, 2, 1), (320, 320, 15, 2), (600, 640, 30, 4))],
    # float32, few rows of the hidden state, four at a time: one to eight, reductions of both lengths that end inside a step
    # and that leave wavefronts without one, one round of phase Q and two
    *[(config(f"ll_few_f32_k{h}_{hp}_{B}_{c}", dtype="fp32", h_joint=h, h_pred=hp, B=B), dict(n_clusters=c))
      for h, hp, B, c in ((8, 8, 1, 1), (40, 616, 3, 1), (640, 632, 4, 1), (104, 640, 5, 1), (616, 24, 8, 1), (640, 640, 28, 4), (632, 640, 12, 4),
                          (256, 248, 8, 1), (48, 248, 80, 16), (240, 200, 128, 16))],
    # ... the shorter reductions, three column tiles a workgroup, four and two rounds, one row to four; and what sixteen rows at a
    # time stay for, two tiles and five rows
    *[(config(f"ll_few_f32_short_k{h}_{hp}_{B}_{c}", dtype="fp32", h_joint=h, h_pred=hp, B=B), dict(n_clusters=c))
      for h, hp, B, c in ((192, 192, 12, 12), (192, 184, 48, 12), (184, 192, 34, 17), (48, 248, 64, 16), (16, 200, 42, 21), (192, 192, 24, 8),
                          (192, 192, 60, 12))],
    # float32, nine to sixteen hypotheses a group and two rounds of phase Q: reductions of both lengths, a second round of one tile and of all
    *[(config(f"ll_f32_rows_k{h}_{hp}_{B}_{c}", dtype="fp32", h_joint=h, h_pred=hp, B=B), dict(n_clusters=c))
      for h, hp, B, c in ((640, 640, 40, 4), (640, 632, 64, 4), (584, 328, 45, 5), (48, 248, 150, 16), (256, 256, 208, 16), (40, 200, 230, 20),
                          (240, 192, 300, 32))],
    # a stateless group of one workgroup by the size of the output layer, and one column beyond
    *[(config(f"ll_one_wg{v}", dtype="fp32", pred_kind="stateless", h_pred=24, vocab=v, B=300), {}) for v in (63, 64)],
    # the form of eight wavefronts: row tiles in pairs and one left over, columns that are no multiple of a
    # batch, workgroups without columns, packed rows, the longest reduction, durations in the last columns
    *[(config(f"ll_wide{w}_{B}_{v}", vocab=v, durations=d, B=B, pred_layers=n, h_joint=h), dict(n_clusters=4, window=w, joint_kernel=2))
      for w, B, v, d, n, h in ((4, 16, 1100, (0, 1, 2), 1, 48), (8, 16, 1023, (), 2, 264), (5, 36, 3000, (1, 2), 2, 1024),
                               (64, 8, 40, (0, 1), 1, 8), (3, 44, 500, (), 1, 1000))],
    # more than eight hypotheses in a row tile, as many batches as there are buffers and one more or less
    *[(config(f"ll_wide_rows_{k}{n}_{v}", pred_kind=k, pred_layers=n, emb_dim=24, h_pred=hp, vocab=v, B=64, h_joint=h, durations=(0, 1)),
       dict(n_clusters=4, window=w, joint_kernel=2))
      for k, n, hp, v, h, w in (("lstm", 1, 40, 120, 1000, 1), ("lstm", 2, 104, 700, 72, 2), ("stateless", 2, 48, 3000, 616, 1),
                                ("lstm", 1, 40, 2000, 1024, 1), ("stateless", 1, 24, 4090, 104, 3))],
    # ... the predictor's column tiles as lists: as many as there is room for and more, some workgroups without any, one layer to
    # four, reductions of three steps a wavefront and of four, one row tile and several
    *[(config(f"ll_wide_lists_{hp}_{n}_{B}_{c}", h_pred=hp, pred_layers=n, vocab=700, B=B, T=14, len_hi=14, durations=(0, 1, 2)),
       dict(n_clusters=c, joint_kernel=2))
      for hp, n, B, c in ((640, 2, 64, 16), (768, 1, 40, 32), (776, 2, 40, 32), (1024, 3, 24, 16), (1000, 1, 70, 4), (40, 4, 150, 4),
                          (648, 2, 100, 32), (16, 1, 3, 4), (1000, 1, 140, 8), (264, 1, 60, 16))],
    # ... one layer and one round of them: six tiles a workgroup and one, workgroups without any, packed rows, one row tile and several
    *[(config(f"ll_wide_round_k{h}_{hp}_{B}_{c}", h_joint=h, h_pred=hp, vocab=700, B=B, T=14, len_hi=14, durations=(0, 1, 2)),
       dict(n_clusters=c, joint_kernel=2))
      for h, hp, B, c in ((48, 640, 3, 8), (48, 640, 40, 8), (1024, 1000, 70, 4), (1000, 776, 4, 4), (48, 16, 3, 4), (264, 72, 250, 4), (640, 264, 130, 8))],
    (config("ll_wide_stateless", pred_kind="stateless", pred_layers=2, h_pred=48, vocab=700, B=40), dict(n_clusters=4, joint_kernel=2)),
    # deeper LSTMs on several row tiles
    (config("ll_deep", pred_layers=3, B=40), dict(n_clusters=2)),
]


@pytest.mark.parametrize("cfg,opts", CASES, ids=[c.name for c, _ in CASES])
def test_label_loop(oracle_lib, gpu, cfg, opts):   # noqa: F811
    check(oracle_lib, gpu, cfg, max_replayed_frac=0.1, **opts)


@pytest.mark.parametrize("kw", [dict(B=6), dict(B=6, dtype="fp32"), dict(B=40, pred_layers=2), dict(B=9, pred_kind="stateless", h_pred=24),
                                dict(B=20, pred_kind="stateless", h_pred=24, vocab=1000)],
                         ids=["one_layer", "one_layer_f32", "two_layers", "stateless", "stateless_items"])
def test_label_loop_chunks(oracle_lib, gpu, kw):   # noqa: F811
    from test_gpu_chunks import check_chunks
    cfg = config("ll_chunks", durations=(0, 1, 5), **kw)
    for ncl in (0, 1):
        check_chunks(oracle_lib, gpu, cfg, "random", 4, n_clusters=ncl)
    check_chunks(oracle_lib, gpu, cfg, "single", 0)


@pytest.mark.parametrize("kw,ncl", [
    # more than one round of phase Q's tiles a workgroup: six and five of four, four of two
    (dict(B=32, h_pred=320), 16), (dict(B=30, h_pred=248, dtype="fp32"), 16), (dict(B=30, h_pred=320, dtype="fp32"), 10),
    # the longer reductions: one round and two
    (dict(B=15, h_pred=648, h_joint=648), 2), (dict(B=9, h_pred=648, h_joint=648), 3),
    # a row tile of five to eight hypotheses, staged as planes, and a full one
    (dict(B=8, h_pred=96), 1), (dict(B=13, h_pred=96), 1), (dict(B=16, h_pred=640, h_joint=640), 2),
    # float32, more than eight hypotheses a group: two rounds with reductions of both lengths, and one round
    (dict(B=40, h_pred=640, h_joint=640, dtype="fp32"), 4), (dict(B=64, h_pred=640, h_joint=640, dtype="fp32"), 4),
    (dict(B=150, h_pred=248, dtype="fp32"), 16), (dict(B=26, h_pred=328, h_joint=328, dtype="fp32"), 2), (dict(B=13, h_pred=96, dtype="fp32"), 1)],
    ids=["two_rounds", "fp32_two_rounds", "fp32_two_rounds_long", "long", "long_two_rounds", "planes", "full_tile", "planes_640",
         "fp32_rows_long", "fp32_rows_long_full", "fp32_rows", "fp32_rows_long_one_round", "fp32_rows_one_round"])
def test_label_loop_chunks_of_one_layer(oracle_lib, gpu, kw, ncl):   # noqa: F811
    """The state that a chunk takes up and leaves, in the forms of one LSTM layer."""
    from test_gpu_chunks import check_chunks
    cfg = config("ll_chunks1", durations=(0, 1, 5), T=20, len_hi=20, **kw)
    check_chunks(oracle_lib, gpu, cfg, "random", 3, n_clusters=ncl)


@pytest.mark.parametrize("hp,n,B,ncl", [(640, 2, 64, 16), (1024, 3, 24, 16), (1000, 1, 140, 8), (776, 2, 40, 32),   # lists
                                         (1000, 1, 70, 4), (640, 1, 24, 8), (16, 1, 3, 4)])                          # one round
def test_label_loop_chunks_of_eight_wavefronts(oracle_lib, gpu, hp, n, B, ncl):   # noqa: F811
    """The state that a chunk takes up and leaves where the predictor's column tiles are lists -- of more tiles than there is room
    for, reductions of three steps a wavefront and of four, one row tile and several -- and where they are one round, packed rows
    and workgroups without tiles among them."""
    from test_gpu_chunks import check_chunks
    cfg = config(f"ll_wide_chunks_{hp}_{n}_{B}", h_pred=hp, pred_layers=n, vocab=700, B=B, T=14, len_hi=14, durations=(0, 1, 2))
    check_chunks(oracle_lib, gpu, cfg, "random", 3, n_clusters=ncl, joint_kernel=2)


# ------------------------------------------------------------------ hypotheses that do not wait for all searches
MERGED = {
    # rows of a group of one layer: packed planes, pairs, a full tile; two rounds of phase Q; workgroups without a work item
    # in some passes; no predictor.  Last: blank biases of an RNN-T, a TDT and a multi-blank model with a label on every second to tenth frame
    "packed": (dict(B=40), dict(n_clusters=10), (3.0, 2.5, 2.5)),
    "pairs": (dict(B=70, h_joint=616, h_pred=96), dict(n_clusters=10), (3.0, 2.5, 2.5)),
    "full_tile": (dict(B=32, h_joint=640, h_pred=200), dict(n_clusters=2), (4.0, 3.5, 2.5)),
    "two_rounds": (dict(B=96, h_pred=320), dict(n_clusters=16), (4.0, 3.0, 1.5)),
    "few_columns": (dict(B=120, vocab=150), dict(n_clusters=30), (3.0, 2.5, 2.0)),
    "fp32": (dict(B=30, dtype="fp32", h_joint=264), dict(n_clusters=3), (3.0, 2.5, 2.5)),
    "stateless": (dict(B=40, pred_kind="stateless", pred_layers=2, h_pred=48), dict(n_clusters=8), (2.5, 2.5, 2.5)),
    "stateless_long": (dict(B=60, pred_kind="stateless", h_pred=24, h_joint=648), dict(n_clusters=3), (3.5, 3.5, 2.5)),
    # the predictor's rows read from the exchange buffers in every pass: longer reductions, deeper LSTMs on one row tile and
    # on two, eight wavefronts
    "fed": (dict(B=30, h_joint=648), dict(n_clusters=3), (3.0, 2.5, 2.0)),
    "fed_two_rounds": (dict(B=30, h_joint=648, h_pred=648), dict(n_clusters=4), (3.0, 2.5, 2.0)),
    "deep": (dict(B=96, pred_layers=2), dict(n_clusters=4), (2.0, 1.5, 2.0)),
    "deep_tiles": (dict(B=60, pred_layers=3, h_pred=104), dict(n_clusters=3), (4.5, 4.0, 2.5)),
    "deep_fp32": (dict(B=64, dtype="fp32", pred_layers=2, h_joint=264), dict(n_clusters=3), (3.0, 2.5, 2.0)),
    "wide": (dict(B=40, pred_layers=2, h_joint=264), dict(n_clusters=4, joint_kernel=2), (3.5, 3.0, 2.0)),
    "wide_stateless": (dict(B=44, pred_kind="stateless", h_pred=24), dict(n_clusters=4, joint_kernel=2), (4.0, 4.0, 3.0)),
}


@pytest.mark.parametrize("kind", MERGED)
def test_a_label_does_not_wait_for_every_search(oracle_lib, gpu, kind):   # noqa: F811
    """Searches of several short passes: a hypothesis that has found its label takes its predictor step while others still
    search -- a group then has more predictor steps than its longest hypothesis has labels -- and every hypothesis is the
    oracle's, as a whole and in chunks; with a caller's window the loops are those of Algorithm 3."""
    from test_gpu_chunks import check_chunks
    kw, opts, biases = MERGED[kind]
    kw = dict(dict(vocab=1500, T=100, len_lo=60, len_hi=100), **kw)
    more_steps = 0
    for bias, more in zip(biases, (dict(), dict(durations=(0, 1, 3)), dict(durations=(2, 4), multi_blank=True))):
        cfg = config(f"ll_merged_{kind}_{len(more)}", default_blank_bias=bias, **kw, **more)
        w = synth.generate_model(cfg)
        enc, ln = synth.generate_inputs(cfg)
        out, _ = check(oracle_lib, gpu, cfg, w, enc, ln, max_replayed_frac=0.1, **opts)
        printed, _ = check(oracle_lib, gpu, cfg, w, enc, ln, max_replayed_frac=0.1, window=2, **opts)
        more_steps += out["stats"]["pred_passes"] - printed["stats"]["pred_passes"]
        assert printed["stats"]["outer_max"] in (printed["len"].max(), printed["len"].max() + 1)
    assert more_steps > 0
    check_chunks(oracle_lib, gpu, config(f"ll_merged_{kind}", durations=(0, 1, 5), default_blank_bias=biases[1], **kw), "random", 3, **opts)


# ------------------------------------------------------------------ values that are no numbers
KINDS = {
    "lstm": (dict(B=9), {}),
    "lstm_planes": (dict(B=7), dict(n_clusters=1)),
    "lstm_full_tile": (dict(B=13), dict(n_clusters=1)),
    "lstm_two_rounds": (dict(B=32, h_pred=320), dict(n_clusters=16)),
    "lstm_long": (dict(B=7, h_joint=648, h_pred=648), dict(n_clusters=2)),
    "lstm_groups": (dict(B=33, h_pred=96), dict(n_clusters=1)),
    "lstm_packed": (dict(B=3), dict(n_clusters=1)),
    "deep": (dict(B=9, pred_layers=3), {}),
    "fp32": (dict(B=9, dtype="fp32"), {}),
    "wide": (dict(B=20, vocab=600, durations=(0, 1, 2)), dict(n_clusters=4, joint_kernel=2)),
    "wide_lists": (dict(B=20, pred_layers=2, vocab=600, durations=(0, 1, 2)), dict(n_clusters=4, joint_kernel=2)),
    "stateless": (dict(B=9, pred_kind="stateless", pred_layers=2, h_pred=48), {}),
    "stateless_items": (dict(B=12, pred_kind="stateless", pred_layers=2, h_pred=48, vocab=300), dict(n_clusters=1)),
    "stateless_eight": (dict(B=12, pred_kind="stateless", pred_layers=2, h_pred=48, vocab=1000), dict(n_clusters=12, joint_tiles=8)),
    "stateless_fp32": (dict(B=9, dtype="fp32", pred_kind="stateless", h_pred=24), {}),
}


@pytest.mark.parametrize("kind", KINDS)
def test_values_that_are_no_numbers(oracle_lib, gpu, kind):   # noqa: F811
    """NaN in valid frames and in what one label puts into the predictor (a NaN gate stays in the state:
    from that label on the joint network sees the encoder alone), masks of minus infinity and of the
    type's lowest value in the output bias: the oracle's hypotheses.  Infinite frames, whose logits are
    not all numbers: what the general kernel gives."""
    kw, opts = KINDS[kind]
    cfg = config(f"ll_nan_{kind}", **kw)
    w = synth.generate_model(cfg)
    enc, ln = synth.generate_inputs(cfg)
    ln[0] = cfg.T
    rng = np.random.default_rng(5)
    # the labels that are emitted most, in a clean run: poisoned, the decode has to meet them
    u_cap = cfg.T * cfg.max_symbols
    clean = run_gpu(gpu, cfg, w, enc, ln, u_cap, **opts)
    seen = np.concatenate([clean["labels"][b, :clean["len"][b]] for b in range(cfg.B)])
    labels = np.argsort(np.bincount(seen, minlength=cfg.vocab))[::-1][:3]
    wn = {k: v.copy() for k, v in w.items()}
    emb = wn["emb"].reshape(-1, cfg.vocab + 1, cfg.emb_dim)   # (stateless: one table a context position)
    for k in labels:
        emb[:, k, int(rng.integers(cfg.emb_dim))] = np.nan
    en = enc.copy()
    for b in range(0, cfg.B, 2):
        if ln[b] > 0:
            en[b, int(rng.integers(ln[b])), int(rng.integers(cfg.d_enc))] = np.nan
            en[b, int(rng.integers(ln[b]))] = np.nan
    check(oracle_lib, gpu, cfg, wn, en, ln, **opts)
    wm = {k: v.copy() for k, v in w.items()}
    masked = rng.permutation(cfg.vocab)[:cfg.vocab // 2]
    wm["b_out"][masked[::2]] = -np.inf
    wm["b_out"][masked[1::2]] = np.finfo(np.float32).min
    out, _ = check(oracle_lib, gpu, cfg, wm, enc, ln, **opts)
    for b in range(cfg.B):
        assert not np.isin(out["labels"][b, :out["len"][b]], masked).any()
    ei = enc.copy()
    for b in range(1, cfg.B, 2):
        if ln[b] > 0:
            ei[b, int(rng.integers(ln[b])), :2] = np.inf, -np.inf
    a = run_gpu(gpu, cfg, w, ei, ln, u_cap, **opts)
    g = run_gpu(gpu, cfg, w, ei, ln, u_cap, algorithm=1)   # (frame-looping: the general kernel)
    assert (a["len"] == g["len"]).all()
    for b in range(cfg.B):
        n = a["len"][b]
        assert (a["labels"][b, :n] == g["labels"][b, :n]).all() and (a["frames"][b, :n] == g["frames"][b, :n]).all()


@pytest.mark.parametrize("B,ncl", [(3, 1), (7, 1), (12, 1), (9, 3)])
def test_a_carried_state_of_all_ones(gpu, B, ncl):   # noqa: F811
    """The bit pattern that stands for what is not there yet, as the hidden state a caller hands in (a NaN): nobody waits
    for it, and the other hypotheses' results are what they are without it."""
    import torch
    from paper_2406_06220_amd import binding
    cfg = config(f"ll_ones_{B}_{ncl}", B=B, h_pred=72, T=12, len_lo=12, len_hi=12)
    w = synth.generate_model(cfg)
    enc, _ = synth.generate_inputs(cfg)
    model = gpu.DeviceModel(cfg, w)
    enc_d = model.upload_enc(enc)
    ln = torch.full((B,), 6, dtype=torch.int32, device=model.device)
    outs = []
    for poisoned in (False, True):
        state = binding.StreamState(model, B)
        dec = binding.ChunkDecoder(model, B, 6, 6 * cfg.max_symbols, state, n_clusters=ncl)
        dec(enc_d[:, :6].contiguous(), ln)
        torch.cuda.synchronize()
        if poisoned:
            at = state.ptr - state.buf.data_ptr() + 4 * (-(-4 * B // 256) * 256)
            h = state.buf[at:at + 4 * B * cfg.h_pred].view(torch.int32).view(B, cfg.h_pred)
            h[B // 2] = -1
            h[B - 1, 5:8] = -1
        dec(enc_d[:, 6:].contiguous(), ln)
        outs.append(dec.results())
    clean, out = outs
    assert out["stats"]["abort"] == 0 and not (out["status"] & gpu.TDT_HYP_ABORTED).any()
    for b in range(B):
        if b not in (B // 2, B - 1):
            n = out["len"][b]
            assert n == clean["len"][b] and (out["labels"][b, :n] == clean["labels"][b, :n]).all()


ONES = {
    # one layer in bfloat16, whose hidden state travels as terms: packed, pairs, a full tile, several groups; reductions beyond 640
    **{f"B{B}_{c}": (dict(B=B), dict(n_clusters=c)) for B, c in ((3, 1), (7, 1), (12, 1), (9, 3))},
    "long": (dict(B=7, h_joint=648), dict(n_clusters=1)),
    # float32: rows four at a time, sixteen
    "fp32_few": (dict(B=7, dtype="fp32", h_joint=264), dict(n_clusters=1)),
    "fp32": (dict(B=12, dtype="fp32", h_joint=264), dict(n_clusters=1)),
    # deeper LSTMs, packed rows and not; eight wavefronts
    "deep_packed": (dict(B=4, pred_layers=2), dict(n_clusters=1)),
    "deep": (dict(B=20, pred_layers=2), dict(n_clusters=1)),
    "wide": (dict(B=20, pred_layers=2), dict(n_clusters=4, joint_kernel=2)),
    "wide_round": (dict(B=20), dict(n_clusters=4, joint_kernel=2)),
    "wide_round_packed": (dict(B=6), dict(n_clusters=4, joint_kernel=2)),
}


@pytest.mark.parametrize("kind", ONES)
def test_a_carried_state_of_all_ones_is_taken_up(gpu, kind):   # noqa: F811
    """The bit pattern that stands for what is not there yet, as the hidden state a caller hands in (a NaN): nobody waits
    for it, the hypotheses it was handed to keep a NaN, and the other hypotheses' results are what they are without it."""
    import torch
    from paper_2406_06220_amd import binding
    kw, opts = ONES[kind]
    cfg = config(f"ll_ones_{kind}", h_pred=72, T=12, len_lo=12, len_hi=12, **kw)
    B = cfg.B
    w = synth.generate_model(cfg)
    enc, _ = synth.generate_inputs(cfg)
    model = gpu.DeviceModel(cfg, w)
    enc_d = model.upload_enc(enc)
    ln = torch.full((B,), 6, dtype=torch.int32, device=model.device)
    hit = (B // 2, B - 1)
    outs, ends = [], []
    for poisoned in (False, True):
        state = binding.StreamState(model, B)
        dec = binding.ChunkDecoder(model, B, 6, 6 * cfg.max_symbols, state, **opts)
        dec(enc_d[:, :6].contiguous(), ln)
        torch.cuda.synchronize()
        if poisoned:
            at = state.ptr - state.buf.data_ptr() + 4 * (-(-4 * B // 256) * 256)
            h = state.buf[at:at + 4 * cfg.pred_layers * B * cfg.h_pred].view(torch.int32).view(cfg.pred_layers, B, cfg.h_pred)
            before = state.download()
            assert (h.cpu().numpy() == before["h"].view(np.int32)).all() and before["h"].any()
            assert before["started"].all() and (before["time"] < 6).all()   # all of them bring their state along
            h[:, hit[0]] = -1
            h[:, hit[1], 5:8] = -1
        dec(enc_d[:, 6:].contiguous(), ln)
        outs.append(dec.results())
        ends.append(state.download())
    clean, out = outs
    assert out["stats"]["abort"] == 0 and not (out["status"] & gpu.TDT_HYP_ABORTED).any()
    lost = np.isnan(ends[1]["h"]).any(axis=2).any(axis=0)
    for b in range(B):
        assert lost[b] == (b in hit) and not np.isnan(ends[0]["h"][:, b]).any(), b
        if b not in hit:
            n = out["len"][b]
            assert n == clean["len"][b] and (out["labels"][b, :n] == clean["labels"][b, :n]).all()
            assert (ends[1]["h"][:, b] == ends[0]["h"][:, b]).all() and (ends[1]["c"][:, b] == ends[0]["c"][:, b]).all()


# ------------------------------------------------------------------ waits that run out
@pytest.mark.parametrize("kind,blank_bias,T", [("stateless", 1e4, 15), ("stateless", 1.0, 40), ("lstm", 1.0, 20)])
def test_a_wait_of_the_label_loop_that_runs_out(oracle_lib, gpu, kind, blank_bias, T):   # noqa: F811
    """15 groups of 17 workgroups and 17 hypotheses, 16 row tiles a pass and an output layer of 1024 column
    tiles: the last workgroup has no work item and waits for the others far longer than the microsecond
    it is given.  Every workgroup leaves the kernel, every hypothesis says so -- also where nothing is
    left to do for the others, who never wait in vain (the first case: one pass, no labels) -- and
    the next call on the same workspace is sound."""
    import parity
    import torch
    kw = dict(pred_kind="stateless", pred_layers=1, h_pred=24) if kind == "stateless" else {}
    cfg = config(f"ll_wait_{kind}_{T}", vocab=16383, B=255, T=T, len_lo=T, len_hi=T, max_symbols=2, **kw)
    w = synth.generate_model(cfg, blank_bias)
    enc, ln = synth.generate_inputs(cfg)
    u_cap = cfg.T * cfg.max_symbols
    model = gpu.DeviceModel(cfg, w)
    dec = gpu.Decoder(model, cfg.B, cfg.T, u_cap, window=15, n_clusters=15, joint_kernel=1)
    enc_d, len_d = model.upload_enc(enc), torch.from_numpy(ln).to(model.device)
    dec.options.wait_timeout_us = 1
    parity.announce(f"waits bounded to 1 us, cfg={cfg.name} blank_bias={blank_bias}")
    dec(enc_d, len_d)
    out = dec.results()
    assert out["stats"]["abort"] >= 1 and (out["status"] & gpu.TDT_HYP_ABORTED).all()
    dec.options.wait_timeout_us = 0
    parity.announce("  the next call on the same workspace")
    dec(enc_d, len_d)
    out = dec.results()
    assert out["stats"]["abort"] == 0 and not (out["status"] & gpu.TDT_HYP_ABORTED).any()
    res = parity.compare(oracle_lib, oracle_lib.OracleModel(cfg, w), cfg, enc, ln, out, u_cap, rows=range(0, cfg.B, 17))
    assert res["replayed"] <= 1, res


# ------------------------------------------------------------------ workspaces
def least_workspace(cfg, B, T):
    """Bytes of the general kernel's arrays, each at a multiple of 256: what every call has to have."""
    up = lambda n: -(-n // 256) * 256
    H, Hp, V, rows = cfg.h_joint, cfg.h_pred, cfg.vocab, B + 256
    L = cfg.pred_layers if cfg.pred_kind == "lstm" else 0
    n = 0
    if cfg.dtype == "bf16":   # the fragment-major copies
        frags = lambda tiles, k: tiles * -(-k // 32) * 1024
        n += up(frags(-(-H // 16), cfg.d_enc) + frags(-(-H // 16), Hp) + frags(-(-cfg.n_out // 16), H) +
                max(2 * L - 1, 0) * frags(-(-Hp // 4), Hp))
    n += up(B * T * H * 4) + up(rows * H * 4)
    n += up((V + 1) * 4 * Hp * 4) if L else up(cfg.pred_layers * (V + 1) * H * 4)
    n += up(2 * 1024 * 256 * 8) + 2 * up(4 * rows * 64 * 8)
    n += up(2 * L * rows * Hp * 4) + up(L * rows * Hp * 4) + (up(rows * 4 * Hp * 4) if L else 0)
    return n + up(257 * 32 * 4) + 256


@pytest.mark.parametrize("kw,opts,label_kernel", [
    (dict(B=5, h_pred=320, h_joint=320), {}, True), (dict(B=30, pred_layers=3), {}, True),
    (dict(B=9, vocab=4200, h_joint=200), dict(joint_kernel=2), True),
    (dict(B=40, pred_kind="stateless", h_pred=24), {}, True),
    (dict(B=5, dtype="fp32", h_pred=320, h_joint=320, vocab=3000), {}, False)])
def test_least_workspace(oracle_lib, gpu, kw, opts, label_kernel):   # noqa: F811
    """A workspace without room for float32 copies of the matrices is enough: nothing beyond it is written,
    and a bfloat16 call gives bit for bit what it gives with the size it is asked for.  With less a
    call is refused."""
    import parity
    import torch
    cfg = config("ll_least_ws", **kw)
    w = synth.generate_model(cfg)
    enc, ln = synth.generate_inputs(cfg)
    u_cap = cfg.T * cfg.max_symbols
    model = gpu.DeviceModel(cfg, w)
    dec = gpu.Decoder(model, cfg.B, cfg.T, u_cap, **opts)
    enc_d, len_d = model.upload_enc(enc), torch.from_numpy(ln).to(model.device)
    least = least_workspace(cfg, cfg.B, cfg.T)
    assert least <= dec.ws_bytes
    parity.announce(f"workspace of {least} of {dec.ws_bytes} bytes, cfg={cfg.name} {kw}")
    dec(enc_d, len_d)
    full = dec.results()
    dec.workspace.fill_(0xA5)
    dec.ws_bytes = least
    dec(enc_d, len_d)
    out = dec.results()
    assert out["stats"]["abort"] == 0
    at = dec.ws_ptr - dec.workspace.data_ptr()
    assert (dec.workspace[at + least:] == 0xA5).all() and (dec.workspace[:at] == 0xA5).all()
    if label_kernel:
        for key in ("labels", "frames", "len", "score", "status", "stats"):
            assert np.all(full[key] == out[key]), key
    parity.compare(oracle_lib, oracle_lib.OracleModel(cfg, w), cfg, enc, ln, out, u_cap)
    dec.ws_bytes = least - 256
    with pytest.raises(gpu.TdtError) as e:
        dec(enc_d, len_d)
    assert e.value.code == -5
