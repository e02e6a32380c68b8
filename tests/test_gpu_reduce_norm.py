"""Residual projections with K split, whose reduction applies the RMSNorm that
follows: row widths of one and two chunks per thread with partly idle threads, two
to sixteen slices (part of a batch of four, one whole, and two and four past the
first), one gain (one-pass, last row) and two in a row (recursive), against the
oracle.  That these products are split, and in how many slices, is what
test_gemm_dispatch.py checks on the CPU."""
import numpy as np
import pytest
import torch

from paper_2608_28099_amd import binding, configs, inputs

from .helpers import check_logits, oracle_outputs, oracle_outputs_recursive

pytestmark = pytest.mark.gpu


HEADS, KV_HEADS, HEAD_DIM = 16, 2, 128
# hidden, batch, SwiGLU width, then the K slices of o (both forms) and of fc and
# down (recursive form); 1: not split, its norm is a launch of its own.  Widths of
# one chunk per thread (2624: ends inside a wave) and of two (4160 to 8192)
CASES = [(2624, 66, 2048, 4, 6, 4), (4160, 70, 2048, 3, 5, 3), (4224, 20, 2048, 4, 7, 4), (5120, 20, 5120, 4, 8, 8),
         (8192, 64, 2048, 2, 4, 2), (1024, 33, 8192, 1, 1, 8), (1024, 20, 8192, 1, 1, 16)]


@pytest.mark.parametrize("hidden,batch,intermediate", [c[:3] for c in CASES])
@pytest.mark.parametrize("recursive", [False, True])
def test_norms_in_the_reduction(hidden, batch, intermediate, recursive):
    k = 2 if recursive else 1
    w = configs.Workload(name="rn", dtype="bf16", batch=batch, k=k, hidden=hidden, n_q_heads=HEADS,
                         n_kv_heads=KV_HEADS, head_dim=HEAD_DIM, intermediate=intermediate, n_classes=4,
                         seq_len=("uniform", 0, 40), weight_std=0.02, seed=hidden + batch)
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
