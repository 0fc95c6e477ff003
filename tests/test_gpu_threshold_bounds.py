"""Thresholds of every size that a plan accepts, in the column kernels (which
compare squares) and in the pass kernels: an all-zero group is never flagged,
any group under a boundless threshold neither, every other group under a
vanishing one."""
import numpy as np
import pytest

import tfft_inputs as inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kappa", [1e-300, 1e-120, 1e120, 1e200, 1.7e308])
@pytest.mark.parametrize("group,form", [(0, "columns"), (32, "pass")])
def test_zero_and_random_groups(group, form, kappa):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2405_02520_amd as tf

    n, batch = 1 << 14, 128
    assert set(tf.forms(n, batch, "c64", group=group)) == {form}
    x = torch.from_numpy(inputs.uniform(9900, batch, n, np.complex64)).cuda()
    print(f"threshold {form} kappa={kappa}", flush=True)
    with tf.Plan(n, batch, "c64", group=group, kappa=kappa) as plan:
        groups = sum(plan.info()["groups"])
        for data, flagged in ((torch.zeros_like(x), 0), (x, 0 if kappa > 1 else groups), (x * 1e-30, 0 if kappa > 1 else groups)):
            for inverse in (False, True):
                (plan.inverse if inverse else plan.forward)(data, ft_mode="detect")
                c, _ = plan.report(cap=0)
                # (a rounding residual may be exactly zero)
                assert c["detected"] <= flagged and c["detected"] >= 0.99 * flagged, (inverse, c)
