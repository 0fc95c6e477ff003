"""The column kernels (complex64 passes of 64..512 points, one lane per member
of a 64-member checksum group) against the FP64 oracle: every pass length,
several groups per workgroup (the smallest grid), partial last groups, both
directions, a fault in every pass at every stage, in place, and ragged
classes, whose signals lie where an offset table says."""
import math

import numpy as np
import pytest

import oracle
import tfft_inputs as inputs

pytestmark = pytest.mark.gpu

TOL = 1e-5


@pytest.fixture(scope="module")
def tf():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2405_02520_amd

    return paper_2405_02520_amd


# (log2 n, batch, passes): 64 x 128, 128 x 128, 128 x 256, 256 x 256,
# 256 x 512, 512 x 512, 512 first, and three passes; batches that fill whole
# groups and that do not
CASES = [(13, 67, 0), (14, 32, 0), (15, 21, 0), (16, 9, 0), (17, 7, 0), (18, 5, 0), (18, 4, 0), (20, 3, 0), (21, 2, 0)]


@pytest.mark.parametrize("inverse", [False, True])
@pytest.mark.parametrize("log2n,batch,passes", CASES)
def test_columns_match_oracle(tf, log2n, batch, passes, inverse):
    import torch

    n = 1 << log2n
    x = inputs.uniform(9700 + log2n + batch, batch, n, np.complex64)
    xd = torch.from_numpy(x).cuda()
    ref = oracle.fft(x.astype(np.complex128), inverse=inverse)
    rng = inputs.fault_rng(9700 + log2n)
    print(f"columns 2^{log2n} x {batch} inverse={inverse}", flush=True)
    with tf.Plan(n, batch, "c64", grid_scale=-3) as plan:  # (a grid_scale of its own: no tile launches)
        info = plan.info()
        assert all(g == 64 for g in info["group"])

        def run(mode, out=None):
            y = (plan.inverse if inverse else plan.forward)(xd if out is None else out, out=out, ft_mode=mode)
            return y.cpu().numpy(), *plan.report()

        for mode in ("off", "detect", "correct"):
            y, c, _ = run(mode)
            assert oracle.rel_l2(y, ref) <= TOL and c["detected"] == 0, (mode, c)
        for p in range(info["passes"]):
            done = math.prod(info["pass_len"][: p + 1])
            for stage in range(-1, info["stages"][p]):
                sig, idx = int(rng.integers(batch)), int(rng.integers(n))
                mag = 64.0 * math.sqrt(2.0 * done / 3.0)
                if inverse and p == info["passes"] - 1 and stage == -1:
                    mag /= n  # final values of the inverse carry the 1/N
                plan.set_faults([dict(signal=sig, pass_=p, stage=stage, index=idx, value=mag * (0.6 - 0.8j))])
                y, c, r = run("correct")
                assert c["detected"] == 1 and c["corrected"] == 1, (p, stage, c, r)
                assert (r[0].signal, r[0].pass_, r[0].sub) == (sig, p, idx // info["pass_len"][p])
                assert r[0].method == tf.LOC_QUOTIENT and oracle.rel_l2(y, ref) <= TOL
                y, c, d = run("detect")  # located by the reader of the report
                assert (d[0].signal, d[0].sub, d[0].member, d[0].method) == (sig, r[0].sub, r[0].member, tf.LOC_QUOTIENT)
                # sums and threshold to rounding (of the order of the threshold over kappa)
                assert abs(d[0].residual - r[0].residual) <= d[0].threshold
        plan.set_faults([])
        z, c, _ = run("off", out=xd.clone())  # in place
        assert oracle.rel_l2(z, ref) <= TOL


def test_columns_two_faults_far_apart(tf):
    """Faults in the first and the last group of a workgroup's walk and a
    non-finite value, located per signal."""
    import torch

    n, batch = 1 << 14, 64
    x = inputs.uniform(9800, batch, n, np.complex64)
    with tf.Plan(n, batch, "c64", grid_scale=-3) as plan:
        plan.set_faults([dict(signal=0, pass_=0, stage=-1, index=5, value=complex(float("inf"), 0.0)),
                         dict(signal=63, pass_=0, stage=1, index=n - 1, value=900.0),
                         dict(signal=31, pass_=1, stage=2, index=77, value=5000.0j)])
        y = plan.forward(torch.from_numpy(x).cuda()).cpu().numpy()
        c, r = plan.report()
    assert c["corrected"] == 3 and c["uncorrectable"] == 0, (c, r)
    assert [(q.signal, q.pass_) for q in r] == [(0, 0), (31, 1), (63, 0)]
    assert r[0].method == tf.LOC_PER_SIGNAL
    assert oracle.rel_l2(y, oracle.fft(x.astype(np.complex128))) <= TOL


@pytest.mark.parametrize("log2n,count", [(13, 515), (16, 67), (18, 19), (20, 9)])
def test_columns_ragged_offsets(tf, log2n, count):
    """One length class whose signals lie in reverse order with gaps (more
    wavefronts than a tile launch takes)."""
    import torch

    n = 1 << log2n
    off = (np.arange(count, dtype=np.int64)[::-1] * (n + 6)).copy()
    total = int(off.max()) + n
    x = inputs.uniform_flat(9900 + log2n, total, np.complex64)
    rg = tf.Ragged(np.full(count, n, np.int64), off, "c64")
    d = rg.info()[0][2]
    sig = count - 2
    rg.set_faults([dict(signal=sig, pass_=p, stage=0, index=n // 3,
                        value=64.0 * math.sqrt(2.0 * math.prod(d["pass_len"][: p + 1]) / 3.0)) for p in range(d["passes"])])
    xd = torch.from_numpy(x).cuda()
    out = torch.full_like(xd, 7 + 7j)
    rg.forward(xd, out)
    c, r = rg.report()
    y = out.cpu().numpy()
    assert c["corrected"] == d["passes"] and {q.signal for q in r} == {sig}, (c, r)
    covered = np.zeros(total, bool)
    for i in range(count):
        covered[off[i]:off[i] + n] = True
    assert np.all(y[~covered] == 7 + 7j)
    for i in sorted({0, 1, sig, count - 1, count // 2}):
        assert oracle.rel_l2(y[off[i]:off[i] + n], oracle.fft(x[off[i]:off[i] + n].astype(np.complex128)[None])[0]) <= TOL, i
