"""The order in which the split attention takes its items, over batch sizes at the
edges of the list writer's passes (256 and 1024 sequences) and at the last size that
has a list:
every (sequence, split) is in the list once, and writing it costs time in
proportion to the sequences."""
import numpy as np
import pytest
import torch

from paper_2608_28099_amd import binding, configs, inputs

pytestmark = pytest.mark.gpu

# split_len 256: none to six splits, full last ones, ties and an empty sequence
LENS = (700, 0, 256, 1, 1536, 257, 255, 1025, 256, 1300, 37)


def _probe(batch):
    """A head over eleven stored sequences and a handle for `batch` that repeat them."""
    dev = torch.device("cuda:0")
    w = configs.Workload(name="list", dtype="bf16", batch=len(LENS), k=1, hidden=64, n_q_heads=2, n_kv_heads=1,
                         head_dim=64, intermediate=64, n_classes=2, seq_len=("list", LENS), kv_std=1.5,
                         weight_std=0.1, seed=17)
    return (w, inputs.kv_cache(w, inputs.seq_lens(w), dev), inputs.params(w, dev),
            binding.Probe(w, max_batch=batch, max_seq_len=max(LENS), split_len=256))


def _pick(kv, order):
    idx = torch.as_tensor(order, device=kv.pool.device)
    return inputs.KVCache(kv.pool, kv.block_table[idx].contiguous(), kv.seq_lens[idx].contiguous(), kv.block_size,
                          kv.max_blocks_per_seq, kv.n_kv, kv.head_dim)


@pytest.mark.parametrize("batch", [2, 255, 257, 1023, 1025, 4099, 65534, 65535])
def test_every_split_is_taken_once(batch):
    """A row's attention output does not depend on the batch it comes in, so each
    equals the one of its sequence alone, bit for bit.  A missing item would leave
    the partial that the call before wrote for another sequence."""
    w, kv, params, probe = _probe(batch)
    row = w.n_q_heads * w.head_dim

    def attn(order):
        probe.forward(_pick(kv, order), params)
        tap = probe.tap(binding.SP_TAP_ATTN, len(order), kv.pool.device).view(torch.float16)
        return tap[:len(order) * row].reshape(-1, row)

    alone = torch.cat([attn([i]).clone() for i in range(len(LENS))])
    for order in ([i % len(LENS) for i in range(batch)], [(3 * i + 5) % len(LENS) for i in reversed(range(batch))]):
        assert torch.equal(attn(order), alone[torch.as_tensor(order, device=kv.pool.device)])
    assert probe.check_device_error() == binding.SP_OK
    probe.close()


def test_time_grows_with_the_sequences():
    """Four times the sequences take about four times as long; ranking every pair of
    them took fifteen times as long.  Eight lies between, twofold from either."""
    best = {}
    for batch in (4096, 16384):
        w, kv, params, probe = _probe(batch)
        sub = _pick(kv, np.random.Generator(np.random.PCG64(3)).integers(0, len(LENS), size=batch))
        logits = torch.empty((batch, w.n_classes), dtype=torch.float32, device=kv.pool.device)
        times = []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(4):
                probe.forward(sub, params, logits=logits)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b) / 4)
        best[batch] = min(times)
        probe.close()
    assert best[16384] <= 8 * best[4096], best


def test_split_counts_do_not_crowd_the_memory_channels():
    """Sequences in large contiguous blocks over one or two KV heads.  Nine and thirteen
    equal splits have eight and twelve full ones, which put the same split of every
    sequence on one XCD: against splits of 512 tokens the attention of the slowest took
    1.34 to 1.9 times as long (where the cache lies in memory matters); with the splits
    rotated by the sequence 0.9 to 1.15."""
    dev, worst = torch.device("cuda:0"), {}
    for batch, tokens, n_kv, splits in ((44, 4782, 2, 9), (88, 4782, 1, 9), (30, 8192, 2, 13)):
        w = configs.Workload(name="spread", dtype="bf16", batch=batch, k=2, hidden=512, n_q_heads=4 * n_kv,
                             n_kv_heads=n_kv, head_dim=128, intermediate=768, n_classes=2, seq_len=("fixed", tokens),
                             layout="contiguous", seed=3)
        kv, params = inputs.kv_cache(w, inputs.seq_lens(w), dev), inputs.params(w, dev)
        times = {}
        for split_len in (0, 512):
            probe = binding.Probe(w, split_len=split_len, flags=binding.SP_FLAG_PROFILE)
            assert split_len or probe.plan(batch)["max_splits"] == splits
            for reps in (5, 30):
                for _ in range(reps):
                    probe.forward(kv, params)
                stages, n = probe.profile_read()
            times[split_len] = stages["attention"] / n
            probe.close()
        worst[batch, tokens] = times[0] / times[512]
    assert max(worst.values()) <= 1.25, worst
