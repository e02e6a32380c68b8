"""The rotations of the soft rows at the positions and bases where the reduction
of the angle could go wrong, through the attention output and the logits: long
contexts (angles of 10^5 radians), base 1 (every pair turns by the position), a
base below 1 (angles that grow with the pair), large bases, both head widths
and storage types, rows that do not fill a workgroup's block."""
import numpy as np
import pytest
import torch

from paper_2608_28099_amd import binding, configs, inputs

from .helpers import check_logits, oracle_outputs, oracle_weights

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,hd,base,lens,k,group", [
    ("f32", 64, 10000.0, (70001, 3), 1, 2), ("f32", 128, 1.0, (5000, 0), 5, 1), ("bf16", 128, 0.5, (900, 17), 11, 3),
    ("bf16", 64, 1.0e7, (70003, 16), 3, 4), ("f32", 64, 0.01, (40, 2), 3, 1)])
def test_rotations_match_the_oracle(dtype, hd, base, lens, k, group):
    w = configs.Workload(name="rope", dtype=dtype, batch=len(lens), k=k, hidden=256, n_q_heads=2 * group, n_kv_heads=2,
                         head_dim=hd, intermediate=128, n_classes=6, seq_len=("list", lens), kv_std=2.0,
                         weight_std=0.15, rope_base=base, seed=int(1000 + base % 97 + k))
    dev = torch.device("cuda:0")
    kv, params = inputs.kv_cache(w, inputs.seq_lens(w), dev), inputs.params(w, dev)
    outs = oracle_outputs(w, kv, params, range(w.batch), oracle_weights(params))
    probe = binding.Probe(w)
    check_logits(probe.forward(kv, params).cpu().numpy(), np.stack([o["logits"] for o in outs]), dtype, "logits")
    r = np.stack([o["o"] for o in outs]).reshape(-1)
    t = probe.tap(binding.SP_TAP_ATTN, w.batch, dev).view(torch.float32 if dtype == "f32" else torch.float16)
    # relative 1e-4 (fp32) / 1e-2 (bf16) of the maximum, as every tap
    assert np.max(np.abs(t[:r.size].float().cpu().numpy() - r)) <= (1e-4 if dtype == "f32" else 1e-2) * np.max(np.abs(r))
    probe.close()


def test_work_list_beside_the_rotations_covers_every_sequence():
    """More sequences than one pass of the list's workgroup (256) and than one
    staging of its candidates (1024), at lengths with many ties, in several rounds."""
    w = configs.Workload(name="list", dtype="bf16", batch=1100, k=1, hidden=64, n_q_heads=4, n_kv_heads=2, head_dim=64,
                         intermediate=64, n_classes=3, seq_len=("uniform", 0, 600), weight_std=0.2, seed=77)
    dev = torch.device("cuda:0")
    lens = inputs.seq_lens(w) // 50 * 50
    kv, params = inputs.kv_cache(w, lens, dev), inputs.params(w, dev)
    W = oracle_weights(params)
    probe = binding.Probe(w, split_len=256)
    got = probe.forward(kv, params).cpu().numpy()
    ref = np.stack([oracle_outputs(w, kv, params, [b], W)[0]["logits"] for b in range(w.batch)])
    check_logits(got, ref, "bf16", "logits")
    assert probe.check_device_error() == binding.SP_OK
    probe.close()
