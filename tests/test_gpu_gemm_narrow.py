"""Narrow matrices with long K on 17-128 rows, whose K is split over workgroups:
both sides of the rule's rows and of its K, against the oracle; and the time of
fewer rows against more."""
import numpy as np
import pytest
import torch

from paper_2608_28099_amd import binding, configs, inputs

from .helpers import check_logits, oracle_outputs

pytestmark = pytest.mark.gpu


def _head(batch, hidden, intermediate):
    return configs.Workload(name="narrow", dtype="bf16", batch=batch, k=1, hidden=hidden, n_q_heads=2, n_kv_heads=1,
                            head_dim=64, intermediate=intermediate, n_classes=4, seq_len=("uniform", 0, 40),
                            weight_std=0.02, seed=hidden + batch)


# hidden 128, 1024 (whole 128-column tiles), 192 (64-column tiles only), 96 (neither:
# the row kernel); K of the down projection short (the row kernel) and long, in
# slices of uneven steps of 64, and no multiple of 64 (the row kernel); rows at the edges
@pytest.mark.parametrize("hidden,intermediate", [(128, 2048), (128, 4160), (1024, 8256), (192, 8256), (192, 8224), (96, 4160)])
@pytest.mark.parametrize("batch", [17, 32, 33, 64, 128])
def test_narrow_long_products_match_the_oracle(hidden, intermediate, batch):
    w = _head(batch, hidden, intermediate)
    dev = torch.device("cuda:0")
    kv, params = inputs.kv_cache(w, inputs.seq_lens(w), dev), inputs.params(w, dev)
    rows = sorted({0, 15, 16, batch // 2, batch - 1})
    probe = binding.Probe(w)
    got = probe.forward(kv, params).cpu().numpy()
    outs = oracle_outputs(w, kv, params, rows)
    check_logits(got[rows], np.stack([o["logits"] for o in outs]), "bf16", "logits")
    # residuals after o and down: a few roundings of relative 2^-11
    for tap, key in ((binding.SP_TAP_A, "a"), (binding.SP_TAP_Y, "y")):
        t = probe.tap(tap, batch, dev).view(torch.float32).reshape(batch, 1, hidden).cpu().numpy()[rows]
        r = np.stack([o[key] for o in outs])
        assert np.max(np.abs(t - r)) <= 1e-2 * np.max(np.abs(r)), key
    packed = dict(params, packed=binding.pack_weights(w, params))
    assert np.array_equal(probe.forward(kv, packed).cpu().numpy(), got), "fp16 image"
    assert probe.check_device_error() == binding.SP_OK
    probe.close()


def test_fewer_rows_take_no_longer():
    """1024 x 28672 on 17-64 rows, one workgroup per 16 columns over the whole of K,
    took 52 us where 96 rows took 31."""
    dev, times = torch.device("cuda:0"), {}
    for batch in (17, 32, 64, 96):
        w = _head(batch, 1024, 28672)
        kv, params = inputs.kv_cache(w, inputs.seq_lens(w), dev), inputs.params(w, dev)
        params["packed"] = binding.pack_weights(w, params)
        probe = binding.Probe(w, flags=binding.SP_FLAG_PROFILE)
        for reps in (5, 50):
            for _ in range(reps):
                probe.forward(kv, params)
            stages, n = probe.profile_read()
        times[batch] = stages[binding.STAGES[6]] / n
        probe.close()
    assert all(times[b] <= 1.25 * times[96] for b in (17, 32, 64)), times
