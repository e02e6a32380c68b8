"""Plans of many short attention splits (small batches), whose partials eight
waves fold per query tile: split counts at the edges of the eight waves and of
their four-split batches, ragged lengths with splits past a sequence's end, and
an empty sequence, against the oracle."""
import numpy as np
import pytest
import torch

from paper_2608_28099_amd import binding, configs, inputs

from .helpers import check_logits, oracle_outputs, oracle_weights

pytestmark = pytest.mark.gpu


# split_len 256: 7 splits (one wave folds them), 8, 9, 32, 33 and 41 (a second
# and third batch per wave); 1, 17 and 40 query rows per KV head (a ragged and a
# third tile), head_dim 64 and 128
@pytest.mark.parametrize("lens,k,group,hd", [
    ((1792, 0), 1, 1, 128), ((2048, 255), 1, 4, 128), ((2049, 1), 17, 1, 64), ((8192, 257, 4097), 5, 8, 128),
    ((8193, 0, 2300), 1, 1, 64), ((10300, 8192), 2, 4, 128)])
def test_many_splits_match_the_oracle(lens, k, group, hd):
    w = configs.Workload(name="many_splits", dtype="bf16", batch=len(lens), k=k, hidden=256, n_q_heads=2 * group,
                         n_kv_heads=2, head_dim=hd, intermediate=256, n_classes=4, seq_len=("list", lens),
                         kv_std=1.5, weight_std=0.1, seed=900 + max(lens))
    dev = torch.device("cuda:0")
    kv, params = inputs.kv_cache(w, inputs.seq_lens(w), dev), inputs.params(w, dev)
    probe = binding.Probe(w, split_len=256)
    assert probe.plan(w.batch)["max_splits"] == -(-max(lens) // 256)
    got = probe.forward(kv, params).cpu().numpy()
    outs = oracle_outputs(w, kv, params, range(w.batch), oracle_weights(params))
    check_logits(got, np.stack([o["logits"] for o in outs]), "bf16", "logits")
    # attention output: fp16 roundings of relative 2^-11 (1e-2 of the maximum, as every tap)
    n = w.batch * k * w.n_q_heads * hd
    t = probe.tap(binding.SP_TAP_ATTN, w.batch, dev).view(torch.float16)[:n].float().cpu().numpy()
    r = np.stack([o["o"] for o in outs]).reshape(-1)
    assert np.max(np.abs(t - r)) <= 1e-2 * np.max(np.abs(r))
    assert probe.check_device_error() == binding.SP_OK
    probe.close()


def test_small_batch_plans_and_the_scratch_limit():
    """A single long sequence takes short splits; a config that fits the static
    scratch of the call without a handle only with 1024-token splits keeps them."""
    w = configs.WORKLOADS["long_9b_bf16"].replace(batch=1, seq_len=("fixed", 2048))
    plan = binding.sp_probe_plan_config(binding.make_config(w), 256)
    assert plan["split_len"] == 256 and plan["max_splits"] == 8
    edge = configs.Workload(name="edge", dtype="bf16", batch=50, k=32, hidden=512, n_q_heads=16, n_kv_heads=4,
                            head_dim=128, intermediate=512, n_classes=2, seq_len=("fixed", 1024))
    plan = binding.sp_probe_plan_config(binding.make_config(edge), 256)
    assert plan["split_len"] == 1024 and plan["workspace_bytes"] <= 64 << 20
    # ten sequences more do not fit either way and take the short splits
    plan = binding.sp_probe_plan_config(binding.make_config(edge.replace(batch=60)), 256)
    assert plan["split_len"] == 512 and plan["workspace_bytes"] > 64 << 20
