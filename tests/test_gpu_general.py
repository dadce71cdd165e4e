"""The general kernel of csrc/decode.hip where label_loop.hip's does not run: how it splits a call, against
the oracle."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2406_06220_amd import synth
from test_gpu_parity import check, gpu, run_gpu  # noqa: F401  (gpu: the fixture)

pytestmark = pytest.mark.gpu


def only_blanks(cfg):
    """Every utterance of full length and a blank that always wins: one pass per window of frames."""
    w = synth.generate_model(cfg, 1e4)
    enc, _ = synth.generate_inputs(cfg)
    return w, enc, np.full(cfg.B, cfg.T, np.int32)


@pytest.mark.parametrize("dtype,H", [("bf16", 1032), ("fp32", 648)])
def test_small_output_layer_keeps_its_group(oracle_lib, gpu, dtype, H):   # noqa: F811
    """A stateless model whose reduction label_loop.hip does not hold, with an output layer small enough for
    a workgroup of its own there: here its groups have all workgroups, so that one pass takes 64 frames."""
    cfg = synth.small_config("gen_small_out", dtype=dtype, d_enc=24, h_pred=16, emb_dim=16, h_joint=H, vocab=20, B=3, T=64,
                             len_lo=64, len_hi=64, seed=401, default_blank_bias=0.6)
    check(oracle_lib, gpu, cfg)
    out = run_gpu(gpu, cfg, *only_blanks(cfg), 10)
    assert (out["len"] == 0).all() and out["stats"]["joint_passes_max"] == 1


def test_windows_of_the_general_kernel(oracle_lib, gpu):   # noqa: F811
    """Projections on the fly at config 2's sizes: eight column tiles an item, so seven hypotheses look 11
    frames ahead and six 13 (the label loop's rule gives six and eight), 250 frames in 23 passes."""
    import dataclasses
    cfg = dataclasses.replace(synth.CFG2, name="gen_windows", d_enc=64, emb_dim=64, vocab=1024)
    out = run_gpu(gpu, cfg, *only_blanks(cfg), 10, projections=1)
    assert out["stats"]["joint_passes_max"] == 23


# ------------------------------------------------------------------ the streaming joint pass of this kernel
def streamed(**kw):
    base = dict(dtype="bf16", pred_kind="lstm", d_enc=48, h_pred=56, emb_dim=24, h_joint=72, vocab=700, B=13, T=30, len_lo=0,
                len_hi=30, seed=402, default_blank_bias=1.5, max_symbols=3)
    base.update(kw)
    return synth.small_config("gen_streaming", **base)


@pytest.mark.parametrize("kw,opts", [
    # an LSTM wider than label_loop.hip's reductions: labels and durations in one tile, a last tile that is
    # mostly padding; several row tiles of a pass; a joint width that is no multiple of a chunk, the widest
    (dict(h_pred=1096, vocab=4501, durations=(0, 1, 2, 4)), {}), (dict(h_pred=1032, B=40), dict(window=9, n_clusters=4)),
    (dict(h_pred=1032, h_joint=1000, B=5, T=12, len_hi=12), dict(window=1)), (dict(h_pred=1032, h_joint=1024, B=5, T=12, len_hi=12), {}),
    # more hypotheses a group than it has lanes for
    (dict(B=300, T=14, len_hi=14), dict(n_clusters=4)), (dict(B=270, T=14, len_hi=14, durations=(0, 2)), dict(n_clusters=4, window=64)),
    (dict(B=300, T=14, len_hi=14, pred_kind="stateless", pred_layers=2, h_pred=48), dict(n_clusters=4)),
    (dict(B=270, T=14, len_hi=14, durations=(2, 3), multi_blank=True), dict(n_clusters=4))])
def test_streaming_joint_pass_of_the_general_kernel(oracle_lib, gpu, kw, opts):   # noqa: F811
    check(oracle_lib, gpu, streamed(**kw), joint_kernel=2, **opts)


def test_streaming_joint_pass_of_the_general_kernel_in_chunks(oracle_lib, gpu):   # noqa: F811
    from test_gpu_chunks import check_chunks
    check_chunks(oracle_lib, gpu, streamed(h_pred=1032, durations=(0, 1, 5)), "random", 3, joint_kernel=2)
