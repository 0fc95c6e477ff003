"""Small batches run as tile launches (one narrow tile per workgroup, the
checksum groups' sums split over the tiles): outputs, reports and records
against the FP64 oracle and against the pass kernels, which a plan with a
grid_scale of its own keeps.  Sizes at the edges: single wavefronts, one tile
per group, partial last groups, groups of 48 members, every pass count, both sides of the limit."""
import math

import numpy as np
import pytest

import oracle
import tfft_inputs as inputs

pytestmark = pytest.mark.gpu

TOL = {"c64": 1e-5, "c128": 1e-12}
NPDT = {"c64": np.complex64, "c128": np.complex128}


@pytest.fixture(scope="module")
def tf():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2405_02520_amd

    return paper_2405_02520_amd


# (n, batch, group): the last two lie just within and beyond the checked limit
CASES = [(2, 1, 0), (4, 131, 16), (16, 70, 0), (64, 1, 0), (128, 129, 16), (512, 37, 64), (1024, 65, 0), (2048, 33, 0),
         (4096, 17, 0), (1 << 13, 3, 0), (1 << 15, 1, 32), (1 << 16, 3, 0), (1 << 17, 1, 0), (1 << 21, 1, 0), (1 << 9, 8192, 0),
         (1 << 9, 8256, 0)]


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n,batch,group", CASES)
def test_tiles_match_oracle_and_pass_kernels(tf, dtype, n, batch, group):
    import torch

    rng = inputs.fault_rng(n + batch)
    x = inputs.uniform(8800 + n % 97, batch, n, NPDT[dtype])
    xd = torch.from_numpy(x).cuda()
    rows = sorted({0, batch - 1, *(int(v) for v in rng.integers(batch, size=max(1, min(batch, (1 << 20) // n))))})
    print(f"tiles {dtype} n={n} batch={batch} group={group}", flush=True)
    with tf.Plan(n, batch, dtype, group=group) as plan, tf.Plan(n, batch, dtype, group=group, grid_scale=1) as ref:
        info = plan.info()
        p = int(rng.integers(info["passes"]))
        done = math.prod(info["pass_len"][: p + 1])
        # 64 x the RMS: far above the rounding noise of the group's checksum
        fault = [dict(signal=batch - 1, pass_=p, stage=int(rng.integers(-1, info["stages"][p])), index=n // 3,
                      value=64.0 * math.sqrt(2.0 * done / 3.0) * (0.6 - 0.8j))]
        # clean and faulty executions in turn: each report is its own
        for mode, inverse, faults in [("correct", False, fault), ("off", True, []), ("detect", False, fault),
                                      ("correct", True, []), ("correct", False, fault)]:
            got = []
            for q in (plan, ref):
                q.set_faults(faults)
                y = (q.inverse if inverse else q.forward)(xd, ft_mode=mode)
                got.append((y.cpu().numpy(), *q.report()))
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
            yo = oracle.fft(x[rows].astype(np.complex128), inverse=inverse)
            assert oracle.rel_l2(y[rows], yo) <= TOL[dtype]
            assert oracle.rel_l2(y, yr) <= TOL[dtype]


def test_tile_executions_replay_in_a_graph(tf):
    """Captured executions keep their own reports over replays, with eager
    executions (whose counts move the report's base) in between."""
    import torch

    n, batch = 1 << 14, 6
    x = torch.from_numpy(inputs.uniform(8900, batch, n, np.complex64)).cuda()
    out = torch.empty_like(x)
    with tf.Plan(n, batch, "c64") as plan:
        plan.set_faults([dict(signal=4, pass_=1, stage=-1, index=77, value=900.0j)])
        want = plan.forward(x).clone()
        st = torch.cuda.Stream()
        g = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(g, stream=st):
            plan.forward(x, out, stream=st)
        for rep in range(3):
            out.zero_()
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            c, _ = plan.report()
            assert torch.equal(out, want) and c["detected"] == 1 and c["corrected"] == 1, (rep, c)
            y = plan.forward(x, ft_mode="detect" if rep % 2 else "correct")
            c, r = plan.report()
            assert c["detected"] == 1 and c["corrected"] == 1 - rep % 2 and r[0].signal == 4, (rep, c)
