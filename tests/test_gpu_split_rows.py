"""One-pass plans beyond the tile launches: checksum groups shared by several
workgroups (few groups) or whole, each workgroup beginning at a round of its own.
Outputs, reports and records against the FP64 oracle and against plans whose
grid_scale keeps the groups whole.  Sizes: shares of one tile and of several,
whole groups, partial last groups in the first and in the last share."""
import numpy as np
import pytest

import oracle
import tfft_inputs as inputs

pytestmark = pytest.mark.gpu

TOL = {"c64": 1e-5, "c128": 1e-12}
NPDT = {"c64": np.complex64, "c128": np.complex128}

CASES = [("c64", 4096, 514, 0), ("c64", 4096, 1041, 0), ("c64", 4096, 4111, 0), ("c64", 2048, 4100, 0), ("c64", 1024, 4161, 0),
         ("c64", 1024, 16449, 16), ("c64", 256, 65600, 64), ("c128", 1024, 8321, 0), ("c128", 2048, 4161, 0), ("c128", 4096, 2099, 0),
         ("c128", 512, 16449, 0)]


@pytest.mark.parametrize("dtype,n,batch,group", CASES)
def test_shared_groups_match_oracle_and_whole_groups(dtype, n, batch, group):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2405_02520_amd as tf

    rng = inputs.fault_rng(n + batch)
    x = inputs.uniform(9100 + n % 89, batch, n, NPDT[dtype])
    xd = torch.from_numpy(x).cuda()
    print(f"rows {dtype} n={n} batch={batch} group={group}", flush=True)
    with tf.Plan(n, batch, dtype, group=group) as plan, tf.Plan(n, batch, dtype, group=group, grid_scale=1) as ref:
        info = plan.info()
        hit = sorted({0, batch // 2, batch - 1})  # in three groups
        # 64 x the RMS: far above the rounding noise of the group's checksum
        fault = [dict(signal=s, pass_=0, stage=int(rng.integers(-1, info["stages"][0])), index=(7 * s + 5) % n,
                      value=64.0 * (2.0 * n / 3.0) ** 0.5 * (0.6 - 0.8j)) for s in hit]
        rows = sorted({*hit, 1, *(int(v) for v in rng.integers(batch, size=16))})
        yo = {inv: oracle.fft(x[rows].astype(np.complex128), inverse=inv) for inv in (False, True)}
        for mode, inverse, faults in [("correct", False, fault), ("off", True, []), ("detect", False, fault),
                                      ("correct", True, []), ("correct", False, fault)]:
            got = []
            for q in (plan, ref):
                q.set_faults(faults)
                y = (q.inverse if inverse else q.forward)(xd, ft_mode=mode)
                c, r = q.report()
                got.append((y.cpu().numpy(), c, sorted(r, key=lambda v: v.group)))
            (y, c, r), (yr, cr, rr) = got
            assert c == cr, (mode, c, cr)
            assert [(a.signal, a.sub, a.group, a.pass_, a.member, a.action, a.method) for a in r] == [
                (a.signal, a.sub, a.group, a.pass_, a.member, a.action, a.method) for a in rr]
            for a, b in zip(r, rr):
                # the sums differ by rounding only (of the order of the threshold over kappa)
                assert abs(a.residual - b.residual) <= 2 * a.threshold and abs(a.threshold - b.threshold) <= 1e-6 * b.threshold
            assert c["detected"] == (len(faults) if mode != "off" else 0)
            if mode == "detect" and faults:
                continue
            assert c["uncorrectable"] == 0
            assert oracle.rel_l2(y[rows], yo[inverse]) <= TOL[dtype]
            assert oracle.rel_l2(y, yr) <= TOL[dtype]
