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


# hidden 2624: 41 steps of 64 and ragged in tiles of 96, 128 and 160; SwiGLU of 12416
# rows: 129.3 tiles of 96; 25088 rows: 261.3 of 96 (two rounds), 156.8 of 160
@pytest.mark.parametrize("intermediate,batch", [(6208, 9), (6208, 16), (6208, 31), (6208, 64), (6208, 65), (6208, 128),
                                                (12544, 5), (12544, 14), (12544, 32), (12544, 50), (12544, 97),
                                                (12544, 129), (12544, 256)])
def test_streaming_tiles_match_the_oracle(intermediate, batch):
    w = configs.Workload(name="stream", dtype="bf16", batch=batch, k=1, hidden=2624, n_q_heads=34, n_kv_heads=2,
                         head_dim=128, intermediate=intermediate, n_classes=4, seq_len=("uniform", 0, 40),
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
