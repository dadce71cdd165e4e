"""The encoder projection where its kernels meet: around the tile edges of the kernel for small products
(64 x 64 output tiles, K tiles in fours), and the products just below and above the sizes at which the
128 x 128 tiles take over -- against the oracle."""
from __future__ import annotations

import numpy as np
import pytest

import parity
from paper_2406_06220_amd import synth
from test_gpu_parity import check, gpu  # noqa: F401  (gpu: the fixture)

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


# few row tiles, on both sides of where they are given to the dies in order: bfloat16's 64 x 64 tiles, 128 x 128 tiles, float32's
@pytest.mark.parametrize("dtype,rows,d_enc,H", [
    ("bf16", 1472, 72, 72), ("bf16", 1473, 72, 72), ("bf16", 2944, 40, 1000), ("bf16", 2945, 40, 1000),
    ("fp32", 1472, 24, 200), ("fp32", 1473, 24, 200),
    ("bf16", 128, 72, 200), ("bf16", 129, 72, 200), ("bf16", 512, 40, 1272), ("bf16", 513, 40, 1272), ("bf16", 768, 40, 1272),
    ("bf16", 769, 40, 1272), ("bf16", 1535, 40, 2040), ("bf16", 2944, 24, 2040), ("bf16", 2945, 24, 2040),
    ("fp32", 100, 40, 2040), ("fp32", 600, 40, 1272), ("fp32", 1472, 24, 2040), ("fp32", 1473, 24, 2040)])
def test_projection_of_few_row_tiles(oracle_lib, gpu, dtype, rows, d_enc, H):   # noqa: F811
    import torch
    cfg = synth.small_config("projfew", dtype=dtype, d_enc=d_enc, h_joint=H, seed=49, B=1, T=rows, len_lo=rows, len_hi=rows)
    w = synth.generate_model(cfg)
    w["b_enc"] = np.random.default_rng(12).standard_normal(H).astype(np.float32)
    enc, _ = synth.generate_inputs(cfg)
    parity.announce(f"tdt_encoder_projection dtype={dtype} rows={rows} d_enc={d_enc} H={H}")
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


# valid frames in 256 x 256 tiles that stay in a workgroup's hands: one K tile and less, K tiles that are not whole,
# one and several rounds of tiles, column tiles that the workgroups of a die are no multiple of, more utterances than threads
@pytest.mark.parametrize("B,T,lo,d_enc,H", [
    (20, 820, 820, 8, 1024), (20, 820, 300, 64, 1024), (41, 534, 0, 72, 768), (7, 3200, 1000, 136, 768), (64, 640, 0, 128, 256),
    (300, 44, 0, 200, 1280), (530, 40, 3, 64, 1536), (23, 900, 899, 264, 1024)])
def test_projection_large_tiles(oracle_lib, gpu, B, T, lo, d_enc, H):   # noqa: F811
    import torch
    cfg = synth.small_config("projlarge", dtype="bf16", d_enc=d_enc, h_joint=H, seed=48, B=B, T=T, len_lo=lo, len_hi=T)
    assert B * T >= 32768 or -(-B * T // 256) * (H // 256) >= 256, "these shapes are there for the large tiles"
    w = synth.generate_model(cfg)
    w["b_enc"] = np.random.default_rng(9).standard_normal(H).astype(np.float32)
    enc, _ = synth.generate_inputs(cfg)
    ln = np.random.default_rng(10).integers(lo, T + 1, size=B).astype(np.int32)
    ln[B // 2] = T
    if lo == 0:
        ln[[0, 1, B - 1]] = 0
    parity.announce(f"tdt_encoder_projection_valid B={B} T={T} d_enc={d_enc} H={H}")
    model = gpu.DeviceModel(cfg, w)
    enc_d = model.upload_enc(enc)
    valid = torch.arange(T)[None] < torch.from_numpy(ln)[:, None]
    enc_d.view(torch.bfloat16)[~valid.to(enc_d.device)] = float("nan")
    out = torch.full((B * T + 3, H), 7.0, dtype=torch.float32, device=model.device)
    len_d = torch.from_numpy(ln).to(model.device)
    gpu.tdt_encoder_projection_valid(enc_d.data_ptr(), len_d.data_ptr(), B, T, model.c,
                                     out.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    rows = np.flatnonzero(valid.numpy().reshape(-1))
    # every frame of the first, the middle and the last utterances, a draw of the others
    some = np.unique(np.concatenate([rows[:600], rows[-600:], np.random.default_rng(11).choice(rows, min(3000, rows.size), False)]))
    om = oracle_lib.OracleModel(cfg, w)
    flat = enc.reshape(B * T, d_enc)
    ref = np.stack([om.enc_proj_frame(flat[r]) for r in some])
    np.testing.assert_allclose(got[some], ref, atol=2e-4, rtol=1e-5)
    assert np.isfinite(got[rows]).all()
    rest = np.setdiff1d(np.arange(B * T + 3), rows)
    assert (got[rest] == 7.0).all(), "rows that are no valid frame were written"


# on both sides of where 256 x 256 tiles begin: all rows (40 and 39 row tiles, four column tiles), and half-padded utterances (64 and
# 63), one column tile of 32768 rows and one less
@pytest.mark.parametrize("B,T,lo,d_enc,H", [
    (1, 9985, None, 40, 1024), (1, 9984, None, 40, 1024), (16, 1023, 100, 40, 1024), (16, 1008, 100, 40, 1024), (32, 1024, 100, 40, 256),
    (7, 4681, 400, 40, 256)])
def test_projection_where_large_tiles_begin(oracle_lib, gpu, B, T, lo, d_enc, H):   # noqa: F811
    import torch
    cfg = synth.small_config("projbegin", dtype="bf16", d_enc=d_enc, h_joint=H, seed=51, B=B, T=T, len_lo=T, len_hi=T)
    w = synth.generate_model(cfg)
    w["b_enc"] = np.random.default_rng(13).standard_normal(H).astype(np.float32)
    enc, _ = synth.generate_inputs(cfg)
    ln = np.random.default_rng(14).integers(lo or T, T + 1, size=B).astype(np.int32)
    parity.announce(f"projection B={B} T={T} d_enc={d_enc} H={H} lengths from {lo}")
    model = gpu.DeviceModel(cfg, w)
    enc_d, len_d = model.upload_enc(enc), torch.from_numpy(ln).to(model.device)
    out = torch.full((B * T + 3, H), 7.0, dtype=torch.float32, device=model.device)
    stream = torch.cuda.current_stream().cuda_stream
    if lo is None:
        gpu.tdt_encoder_projection(enc_d.data_ptr(), B * T, model.c, out.data_ptr(), stream)
    else:
        gpu.tdt_encoder_projection_valid(enc_d.data_ptr(), len_d.data_ptr(), B, T, model.c, out.data_ptr(), stream)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    valid = np.append((np.arange(T)[None] < ln[:, None]).reshape(-1), [False] * 3)
    rows = np.flatnonzero(valid)
    some = np.unique(np.concatenate([rows[:300], rows[-300:], np.random.default_rng(15).choice(rows, min(2000, rows.size), False)]))
    om = oracle_lib.OracleModel(cfg, w)
    flat = enc.reshape(B * T, d_enc)
    ref = np.stack([om.enc_proj_frame(flat[r]) for r in some])
    np.testing.assert_allclose(got[some], ref, atol=2e-4, rtol=1e-5)
    assert np.isfinite(got[rows]).all() and (got[~valid] == 7.0).all()


# the preparation launch: a projection of 17 or 18 row tiles in order, whose workgroups are no multiple of the dies, ahead of
# per-label tables of 24 row tiles, which are dealt -- one of an LSTM (grouped columns), two of a stateless predictor
@pytest.mark.parametrize("kw", [
    dict(dtype="bf16", pred_kind="lstm", h_pred=160, emb_dim=24, h_joint=640, vocab=3071, B=7, T=311),
    dict(dtype="bf16", pred_kind="stateless", pred_layers=2, h_pred=48, emb_dim=24, h_joint=640, vocab=3071, B=7, T=311),
    dict(dtype="fp32", pred_kind="lstm", h_pred=80, emb_dim=24, h_joint=320, vocab=1535, B=4, T=260),
    dict(dtype="fp32", pred_kind="stateless", pred_layers=2, h_pred=48, emb_dim=24, h_joint=320, vocab=1535, B=4, T=260)])
def test_tiles_in_order_ahead_of_tiles_that_are_dealt(oracle_lib, gpu, kw):   # noqa: F811
    tile = 128 if kw["dtype"] == "bf16" else 64
    ahead = -(-kw["B"] * kw["T"] // tile) * (kw["h_joint"] // tile)
    assert ahead % 8 != 0 and -(-kw["B"] * kw["T"] // tile) in (17, 18) and (kw["vocab"] + 1) // tile == 24
    cfg = synth.small_config("projahead", d_enc=32, len_lo=kw["T"] // 2, len_hi=kw["T"], seed=50, default_blank_bias=4.0, **kw)
    w = synth.generate_model(cfg)
    enc, ln = synth.generate_inputs(cfg)
    check(oracle_lib, gpu, cfg, w, enc, ln, max_replayed_frac=0.2)
