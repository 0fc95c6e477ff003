"""The launch forms that plans are given (host side, no device): both sides of
each line, and the sizes that the GPU tests of a form rely on."""
import ctypes

import pytest


@pytest.fixture(scope="module")
def tf():
    import paper_2405_02520_amd

    return paper_2405_02520_amd


FORMS = [
    # tiles: few wavefronts in every pass, and signals of up to 16 points at any batch
    (dict(n=256, batch=64), ["tile"]),
    (dict(n=16, batch=1 << 20), ["tile"]),
    (dict(n=1 << 14, batch=5), ["tile"] * 2),
    (dict(n=512, batch=16384), ["tile"]),
    (dict(n=512, batch=16448), ["turns"]),
    (dict(n=1024, batch=4096), ["tile"]),
    (dict(n=1024, batch=4160), ["turns"]),
    (dict(n=1024, batch=12288, dtype="c128"), ["tile"]),
    (dict(n=1024, batch=12352, dtype="c128"), ["turns"]),
    (dict(n=4096, batch=2048, dtype="c128"), ["tile"]),
    (dict(n=4096, batch=2064, dtype="c128"), ["pass or turns"]),  # shared where a device is there to fill
    (dict(n=1 << 15, batch=1, passes=3), ["tile"] * 3),
    (dict(n=1 << 16, batch=3, passes=3, dtype="c128"), ["tile"] * 3),
    (dict(n=1 << 21, batch=1), ["pass", "columns", "pass"]),
    # ... that a launch of one workgroup per group holds (less than 2^32 threads)
    (dict(n=2, batch=(1 << 32) - 512), ["tile"]),
    (dict(n=2, batch=(1 << 32) - 511), ["pass"]),
    (dict(n=4, batch=1 << 32, dtype="c128"), ["pass"]),
    # not where the plan has a launch or a scheme of its own
    (dict(n=256, batch=64, grid_scale=1), ["pass"]),
    (dict(n=256, batch=64, scheme="signal"), ["pass"]),
    (dict(n=1 << 14, batch=128, chunk=64), ["columns"] * 2),
    (dict(n=4, batch=131, group=16), ["pass"]),
    # columns: complex64, 64..512 points, whole groups of 64
    (dict(n=1 << 13, batch=1 << 14), ["columns"] * 2),
    (dict(n=1 << 13, batch=1 << 14, dtype="c128"), ["pass"] * 2),
    (dict(n=1 << 13, batch=1 << 14, group=32), ["pass"] * 2),
    (dict(n=1 << 13, batch=1 << 14, scheme="thread", ft_mode="off"), ["columns"] * 2),
    (dict(n=1 << 19, batch=128), ["columns", "pass"]),
    (dict(n=1 << 22, batch=32), ["columns"] * 3),
    # classes of the ragged column tests
    (dict(n=1 << 13, batch=515), ["columns"] * 2),
    (dict(n=1 << 16, batch=67), ["columns"] * 2),
    (dict(n=1 << 18, batch=19), ["columns"] * 2),
    (dict(n=1 << 20, batch=9), ["columns"] * 3),
]


@pytest.mark.parametrize("args,want", FORMS)
def test_forms(tf, args, want):
    got = tf.forms(**args)
    assert len(got) == len(want) and all(g in w.split(" or ") for g, w in zip(got, want)), got


def test_forms_rejects_what_the_plan_rejects(tf):
    out = (ctypes.c_int32 * 3)()
    assert tf.tfft_plan_forms(12, 4, 0, None, 0, out) == tf.E_INVALID
    assert tf.tfft_plan_forms(16, 4, 0, None, 3, out) == tf.E_INVALID
    assert tf.tfft_plan_forms(16, 4, 0, None, 0, None) == tf.E_INVALID
    opt = tf.tfft_options(passes=2)
    assert tf.tfft_plan_forms(1 << 21, 4, 0, ctypes.byref(opt), 0, out) == tf.E_UNSUPPORTED
