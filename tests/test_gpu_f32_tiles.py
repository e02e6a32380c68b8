"""The fp32 path's matrix-core kernels at the edges of their tiles, against the
oracle: widths that are multiples of 4 only (K and column remainders), fewer K
steps than waves, one to four query tiles, 16-row and 64-row projection tiles,
splits shorter than the waves' steps, large blocks, NaN past every end."""
import numpy as np
import pytest
import torch

from paper_2608_28099_amd import binding, configs, inputs

from .helpers import check_logits, oracle_outputs, oracle_weights

pytestmark = pytest.mark.gpu


# (hidden, intermediate, query heads, KV heads, head_dim, k, lengths, layout, block size)
CASES = [
    (36, 52, 2, 2, 64, 1, (0, 1, 15), "paged", 16),
    (100, 4, 4, 1, 64, 16, (16, 17, 255, 256, 257), "paged", 16),        # 64 rows: four tiles
    (60, 300, 17, 1, 128, 1, (129, 700), "contiguous", None),           # 17 rows: a second, nearly empty tile
    (256, 4100, 3, 1, 64, 11, (5, 513, 40), "paged", 64),                # 33 rows; 64-row SwiGLU tiles, remainder
    (4128, 8, 2, 1, 128, 20, (300,), "paged", 32),                       # 64-row o and down tiles, 8 deep
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"d{c[0]}_i{c[1]}_k{c[5]}")
def test_fp32_remainders(case):
    d, inter, nq, nkv, hd, k, lens, layout, bs = case
    w = configs.Workload(name=f"f32_{d}", dtype="f32", batch=len(lens), k=k, hidden=d, n_q_heads=nq, n_kv_heads=nkv,
                         head_dim=hd, intermediate=inter, n_classes=5, seq_len=("list", lens), layout=layout,
                         block_size=bs or 16, kv_std=1.5, weight_std=0.05, seed=d + k)
    dev = torch.device("cuda:0")
    kv, params = inputs.kv_cache(w, inputs.seq_lens(w), dev), inputs.params(w, dev)
    outs = oracle_outputs(w, kv, params, range(w.batch), oracle_weights(params))
    probe = binding.Probe(w)
    got = probe.forward(kv, params).cpu().numpy()
    check_logits(got, np.stack([o["logits"] for o in outs]), "f32", "logits")
    for tap, key in ((binding.SP_TAP_ATTN, "o"), (binding.SP_TAP_A, "a"), (binding.SP_TAP_Y, "y")):
        r = np.stack([o[key] for o in outs]).reshape(-1)
        t = probe.tap(tap, w.batch, dev).view(torch.float32)[:r.size].cpu().numpy()
        # sums of up to 4128 fp32 products: relative 1e-5 of the maximum covers sqrt(4128) roundings of 2^-24
        assert np.max(np.abs(t - r)) <= 1e-5 * np.max(np.abs(r)), key
    assert probe.check_device_error() == binding.SP_OK
    probe.close()
