"""Residual projections with K split, whose reduction applies the RMSNorm that
follows: row widths of one and two chunks per thread with partly idle threads,
one, two and four slices past a four-slice batch, one gain (one-pass, last row)
and two in a row (recursive), against the oracle."""
import numpy as np
import pytest
import torch

from paper_2608_28099_amd import binding, configs, inputs

from .helpers import check_logits, oracle_outputs, oracle_outputs_recursive

pytestmark = pytest.mark.gpu


# 34-256 rows of 128 x 64 tiles: hidden 1024 (8 slices), 2624 (a width that ends
# inside a wave), 4160 (two chunks); 17-32 rows: 32 x 128 tiles, up to 16 slices
@pytest.mark.parametrize("hidden,batch", [(1024, 40), (2624, 66), (4160, 70), (4224, 20)])
@pytest.mark.parametrize("recursive", [False, True])
def test_norms_in_the_reduction(hidden, batch, recursive):
    k = 2 if recursive else 1
    w = configs.Workload(name="rn", dtype="bf16", batch=batch, k=k, hidden=hidden, n_q_heads=16, n_kv_heads=2,
                         head_dim=128, intermediate=2048, n_classes=4, seq_len=("uniform", 0, 40), weight_std=0.02,
                         seed=hidden + batch)
    dev = torch.device("cuda:0")
    kv, params = inputs.kv_cache(w, inputs.seq_lens(w), dev), inputs.params(w, dev)
    rows = [0, 1, batch // 2, batch - 1]
    probe = binding.Probe(w)
    if recursive:
        fusion = inputs.fusion_params(w, dev)
        got = probe.forward_recursive(kv, params, fusion).cpu().numpy()
        outs = oracle_outputs_recursive(w, kv, params, fusion, rows)
    else:
        got = probe.forward(kv, params).cpu().numpy()
        outs = oracle_outputs(w, kv, params, rows)
    check_logits(got[rows], np.stack([o["logits"] for o in outs]), "bf16", "logits")
    # residuals after o and down of every step: a few roundings of relative 2^-11
    for tap, key in ((binding.SP_TAP_A, "a"), (binding.SP_TAP_Y, "y")):
        t = probe.tap(tap, batch, dev).view(torch.float32).reshape(batch, k, hidden).cpu().numpy()[rows]
        r = np.stack([o[key] for o in outs])
        assert np.max(np.abs(t - r)) <= 1e-2 * np.max(np.abs(r)), key
    assert probe.check_device_error() == binding.SP_OK
    probe.close()
