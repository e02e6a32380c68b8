"""The forward without a handle on a static array that holds other calls' bytes:
configs of other shapes and storage types (whose values read as NaN or huge
numbers in the next one's padding) before each, with rows and slots that leave
padding in every buffer; bit for bit the handle's logits."""
import pytest
import torch

from paper_2608_28099_amd import binding, configs, inputs

from .test_zz_no_alloc import noalloc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k,heads,hd,flags", [(1, (4, 4), 128, 0), (3, (10, 2), 64, 0), (33, (4, 2), 128, 0),
                                              (5, (6, 2), 128, binding.SP_FLAG_LAST_ROW_ONLY)])
def test_padding_is_cleared_over_other_contents(k, heads, hd, flags):
    dev = torch.device("cuda:0")
    base = configs.Workload(name="pad", dtype="bf16", batch=3, k=k, hidden=128, n_q_heads=heads[0], n_kv_heads=heads[1],
                            head_dim=hd, intermediate=64, n_classes=4, seq_len=("list", (0, 37, 300)), kv_std=1.5,
                            weight_std=0.1, seed=40 + k)
    # fp32 first (its activations and partials fill the array), then a larger bf16 one
    dirty = [configs.TINY_PEAKY_F32, base.replace(k=64, batch=8, hidden=512, weight_std=3.0,
                                                  seq_len=("uniform", 100, 900), seed=1)]
    lens = inputs.seq_lens(base)
    kv, params = inputs.kv_cache(base, lens, dev), inputs.params(base, dev)
    probe = binding.Probe(base, flags=flags)
    want = probe.forward(kv, params).clone()
    probe.close()
    for w in dirty:
        kd, pd = inputs.kv_cache(w, inputs.seq_lens(w), dev), inputs.params(w, dev)
        out = torch.empty((w.batch, w.n_classes), device=dev)
        assert noalloc(w, kd, pd, w.batch, out) == 0
        got = torch.empty_like(want)
        cfg = binding.make_config(base, flags=flags)
        st = binding.sp_probe_forward_noalloc(cfg, binding.make_kv(kv), kv.seq_lens.data_ptr(), kv.block_table.data_ptr(),
                                              params["soft_prompt"].data_ptr(), binding.make_weights(params),
                                              got.data_ptr(), torch.cuda.current_stream().cuda_stream)
        assert st == 0 and torch.equal(got, want), w.name
