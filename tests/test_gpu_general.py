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
