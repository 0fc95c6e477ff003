"""Setting a plan up costs no more where it runs as tile launches."""
import time

import pytest

pytestmark = pytest.mark.gpu


def test_tile_plans_are_set_up_as_quickly_as_others():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2405_02520_amd as tf

    torch.zeros(1, device="cuda")
    n, batch = 256, 64
    assert tf.forms(n, batch) == ["tile"] and tf.forms(n, batch, grid_scale=1) == ["pass"]
    t = {0: [], 1: []}
    for _ in range(300):  # in turn: clocks and neighbours are the same for both
        for scale in t:
            t0 = time.perf_counter()
            tf.Plan(n, batch, "c64", grid_scale=scale).close()
            t[scale].append(time.perf_counter() - t0)
    tile, plain = (sorted(v)[len(v) // 2] for v in (t[0], t[1]))
    print(f"tile {tile * 1e6:.0f} us, pass kernels {plain * 1e6:.0f} us", flush=True)
    # (57 us each; with tables and buffers of their own tile plans took 158 of 120)
    assert tile <= 1.15 * plain
