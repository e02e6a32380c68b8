"""The projections on at most 16 rows (every compute path of a forward with few
rows) against the oracle: one row up to two packed row groups and past them,
widths that are odd multiples of 32 (uneven slices of K over the waves), the
caller's bf16 matrices and the fp16 image."""
import numpy as np
import pytest
import torch

from paper_2608_28099_amd import binding, configs, inputs

from .helpers import check_logits, oracle_outputs, oracle_weights

pytestmark = pytest.mark.gpu


# batch x k rows past the attention: 1, 7, 8 (packed fragments), 9, 15, 16 (whole
# ones), 18 (the next tile).  hidden 96 and 608, intermediate 32 and 1056: K of
# 1 to 33 steps of 32, fewer than the waves and uneven over them.
@pytest.mark.parametrize("batch,k", [(1, 1), (1, 7), (4, 2), (3, 3), (5, 3), (8, 2), (6, 3)])
@pytest.mark.parametrize("hidden,intermediate", [(96, 32), (608, 1056)])
def test_few_rows_match_the_oracle(batch, k, hidden, intermediate):
    w = configs.SMALL_BF16.replace(name="rows", batch=batch, k=k, hidden=hidden, intermediate=intermediate,
                                   seq_len=("uniform", 0, 90), weight_std=0.05, seed=700 + 10 * batch + k)
    dev = torch.device("cuda:0")
    lens = inputs.seq_lens(w)
    kv, params = inputs.kv_cache(w, lens, dev), inputs.params(w, dev)
    outs = oracle_outputs(w, kv, params, range(batch), oracle_weights(params))
    ref = np.stack([o["logits"] for o in outs])
    probe = binding.Probe(w)
    got = probe.forward(kv, params).cpu().numpy()
    check_logits(got, ref, "bf16", "bf16 matrices")
    # the residuals after o and down, whose rows the logits of LAST do not all show:
    # a few roundings of relative 2^-11 on values of order one (1e-2 of the maximum)
    for tap, key in ((binding.SP_TAP_A, "a"), (binding.SP_TAP_Y, "y")):
        t = probe.tap(tap, batch, dev).view(torch.float32).reshape(batch, k, hidden).cpu().numpy()
        r = np.stack([o[key] for o in outs])
        assert np.max(np.abs(t - r)) <= 1e-2 * np.max(np.abs(r)), key
    packed = dict(params, packed=binding.pack_weights(w, params))
    assert np.array_equal(probe.forward(kv, packed).cpu().numpy(), got), "fp16 image"
    assert probe.check_device_error() == binding.SP_OK
    probe.close()
