"""The encoder projection where its kernels meet: around the tile edges of the kernel for small products
(64 x 64 output tiles, K tiles in fours), and the products just below and above the size at which the
128 x 128 tiles take over -- against the oracle."""
from __future__ import annotations

import numpy as np
import pytest

import parity
from paper_2406_06220_amd import synth
from test_gpu_parity import gpu  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,d_enc,H", [
    (1, 8, 8), (63, 64, 64), (64, 72, 72), (65, 256, 56), (127, 264, 136), (513, 248, 64), (600, 520, 200),
    (20480, 24, 128), (20481, 24, 128), (10240, 40, 256), (10241, 40, 136), (20700, 264, 120)])
def test_projection_tiles(oracle_lib, gpu, rows, d_enc, H):   # noqa: F811
    import torch
    cfg = synth.small_config("projtiles", dtype="bf16", d_enc=d_enc, h_joint=H, seed=47, B=1, T=rows, len_lo=rows, len_hi=rows)
    w = synth.generate_model(cfg)
    w["b_enc"] = np.random.default_rng(8).standard_normal(H).astype(np.float32)
    enc, _ = synth.generate_inputs(cfg)
    parity.announce(f"tdt_encoder_projection rows={rows} d_enc={d_enc} H={H}")
    model = gpu.DeviceModel(cfg, w)
    enc_d = model.upload_enc(enc[0])
    out = torch.full((rows + 3, H), 7.0, dtype=torch.float32, device=model.device)
    gpu.tdt_encoder_projection(enc_d.data_ptr(), rows, model.c, out.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    om = oracle_lib.OracleModel(cfg, w)
    ref = np.stack([om.enc_proj_frame(enc[0, r]) for r in range(rows)])
    np.testing.assert_allclose(got[:rows], ref, atol=2e-4, rtol=1e-5)
    assert (got[rows:] == 7.0).all(), "rows past the end were written"
