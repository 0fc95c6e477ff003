"""Tuning a persistent plan of few short signals keeps what it starts with where
that is the best: 4 tiles per work item."""
import numpy as np
import pytest

import tfft_inputs as inputs

pytestmark = pytest.mark.gpu


def test_tuning_few_signals_does_not_slow_them():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2405_02520_amd as tf

    lengths = np.int64(1) << np.random.default_rng(20240505).integers(8, 17, size=20).astype(np.int64)
    x = torch.from_numpy(inputs.uniform_flat(9950, int(lengths.sum()), np.complex64)).cuda()
    out = torch.empty_like(x)
    rg = tf.Ragged(lengths, dtype="c64", persistent=True)
    st = torch.cuda.Stream()

    def best():
        t = []
        for _ in range(40):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record(st)
            for _ in range(5):
                rg.forward(x, out, use_graph=True, stream=st)
            b.record(st)
            b.synchronize()
            t.append(a.elapsed_time(b) / 5)
        return min(t)

    torch.cuda.synchronize()
    before = best()
    print(f"before {before * 1e3:.1f} us", flush=True)
    rg.tune(x, out, reps=5, stream=st)
    after = best()
    print(f"tuned {after * 1e3:.1f} us", flush=True)
    # (what it starts with is a candidate: 80 us, tuned 64; with 8 tiles per item,
    # formerly the least to choose from, tuned 86)
    assert after <= before
