"""Projections of few rows on the streaming tiles, whose column tiles do not divide
N (the last one is ragged), whose K order differs by column tile and whose K is
split, against the oracle: row counts at the edges of the 16-, 32-, 64- and 128-row
tiles and past them, SwiGLU widths of one round of 96 columns and of 160, the
caller's bf16 matrices and the fp16 image."""
import numpy as np
import pytest
import torch

from paper_2608_28099_amd import binding, configs, inputs

from .helpers import check_logits, oracle_outputs

pytestmark = pytest.mark.gpu


HIDDEN, HEADS, KV_HEADS, HEAD_DIM = 2624, 34, 2, 128
# hidden 2624: 41 steps of 64 and ragged in tiles of 96, 128 and 160; SwiGLU of 12416
# rows: 129.3 tiles of 96; 16640 rows: 173.3 of 96; 25088 rows: 261.3 of 96 (two rounds),
# 156.8 of 160.  The last entry: the SwiGLU's tile, None where it is not a streaming one
# (tests/test_gemm_dispatch.py holds the dispatch to it)
CASES = [(6208, 9, None), (6208, 16, None), (6208, 31, "32x96"), (6208, 64, "64x96"), (6208, 65, None), (6208, 128, None),
         (8320, 9, "16x96"), (8320, 16, "16x96"), (8320, 65, "128x96"), (8320, 128, "128x96"),
         (12544, 5, "16x160"), (12544, 14, "16x160"), (12544, 32, "32x160"), (12544, 50, "64x160"), (12544, 97, "128x160"),
         (12544, 129, None), (12544, 256, None)]


@pytest.mark.parametrize("intermediate,batch", [c[:2] for c in CASES])
def test_streaming_tiles_match_the_oracle(intermediate, batch):
    w = configs.Workload(name="stream", dtype="bf16", batch=batch, k=1, hidden=HIDDEN, n_q_heads=HEADS, n_kv_heads=KV_HEADS,
                         head_dim=HEAD_DIM, intermediate=intermediate, n_classes=4, seq_len=("uniform", 0, 40),
                         weight_std=0.02, seed=intermediate + batch)
    dev = torch.device("cuda:0")
    kv, params = inputs.kv_cache(w, inputs.seq_lens(w), dev), inputs.params(w, dev)
    rows = sorted({0, batch // 2, batch - 1})
    probe = binding.Probe(w)
    got = probe.forward(kv, params).cpu().numpy()
    outs = oracle_outputs(w, kv, params, rows)
    check_logits(got[rows], np.stack([o["logits"] for o in outs]), "bf16", "logits")
    # residuals after o and down: a few roundings of relative 2^-11
    for tap, key in ((binding.SP_TAP_A, "a"), (binding.SP_TAP_Y, "y")):
        t = probe.tap(tap, batch, dev).view(torch.float32).reshape(batch, 1, w.hidden).cpu().numpy()[rows]
        r = np.stack([o[key] for o in outs])
        assert np.max(np.abs(t - r)) <= 1e-2 * np.max(np.abs(r)), key
    packed = dict(params, packed=binding.pack_weights(w, params))
    assert np.array_equal(probe.forward(kv, packed).cpu().numpy(), got), "fp16 image"
    assert probe.check_device_error() == binding.SP_OK
    probe.close()
