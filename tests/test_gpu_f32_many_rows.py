"""The fp32 projections on more rows than one dimension of a launch grid can hold as
16-row tiles (over a million: 16 x 65535), against the oracle."""
import numpy as np
import pytest
import torch

from paper_2608_28099_amd import binding, configs, inputs

from .helpers import check_logits, oracle_outputs

pytestmark = pytest.mark.gpu


def test_a_million_fp32_rows():
    lens, batch, dev = (3, 0, 17, 40), 16400, torch.device("cuda:0")
    w = configs.Workload(name="f32_many", dtype="f32", batch=len(lens), k=64, hidden=32, n_q_heads=1, n_kv_heads=1,
                         head_dim=64, intermediate=36, n_classes=3, seq_len=("list", lens), kv_std=1.5,
                         weight_std=0.1, seed=5)
    kv, params = inputs.kv_cache(w, inputs.seq_lens(w), dev), inputs.params(w, dev)
    ref = np.stack([o["logits"] for o in oracle_outputs(w, kv, params, range(len(lens)))])
    order = [(i * 7 + 1) % len(lens) for i in range(batch)]
    idx = torch.as_tensor(order, device=dev)
    many = inputs.KVCache(kv.pool, kv.block_table[idx].contiguous(), kv.seq_lens[idx].contiguous(), kv.block_size,
                          kv.max_blocks_per_seq, kv.n_kv, kv.head_dim)
    probe = binding.Probe(w, max_batch=batch)
    got = probe.forward(many, params).cpu().numpy()
    check_logits(got, ref[order], "f32", "logits")
    assert probe.check_device_error() == binding.SP_OK
    probe.close()
