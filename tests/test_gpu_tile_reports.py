"""Reports of tile launches, whose flagged groups lie where their records lie:
an execution reads its own whatever ran in between on the same plan."""
import numpy as np
import pytest

import tfft_inputs as inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tf():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2405_02520_amd

    return paper_2405_02520_amd


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n,batch", [(256, 64), (1 << 14, 6)])
def test_reports_with_noalloc_replays_in_between(tf, dtype, n, batch):
    """A captured allocation-free execution (its report in the static scratch)
    replayed after an ordinary one (its report in the plan)."""
    import torch

    npdt = {"c64": np.complex64, "c128": np.complex128}[dtype]
    x = torch.from_numpy(inputs.uniform(9500, batch, n, npdt)).cuda()
    xg, y, out = x.clone(), torch.empty_like(x), torch.empty_like(x)
    bad = x.clone()
    bad[3, 5] = float("nan")  # flags signal 3's groups
    print(f"reports {dtype} {n} x {batch}", flush=True)
    with tf.Plan(n, batch, dtype) as plan:
        st = torch.cuda.Stream()
        g = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(g, stream=st):
            plan.execute_noalloc(xg, out, ft_mode="detect", stream=st)
        for rep in range(3):
            xg.copy_(bad if rep % 2 == 0 else x)
            torch.cuda.synchronize()
            plan.forward(x if rep % 2 == 0 else bad, y, ft_mode="detect")
            g.replay()
            torch.cuda.synchronize()
            c, r = plan.report()  # of the ordinary execution
            assert (c["detected"] > 0) == (rep % 2 == 1), (rep, c)
            assert c["n_records"] == c["detected"] == len(r)
            assert all(v.action == "detected" and 0 <= v.pass_ < plan.info()["passes"] for v in r)
            z = torch.empty_like(x)
            plan.execute_noalloc(bad, z, ft_mode="detect")
            c2, r2 = plan.report()
            plan.execute_noalloc(x, z, ft_mode="detect")
            c3, _ = plan.report()
            assert c2["detected"] > 0 and len(r2) == c2["detected"] and c3["detected"] == 0, (c2, c3)
            if rep % 2 == 1:
                assert [(v.signal, v.pass_, v.group) for v in r] == [(v.signal, v.pass_, v.group) for v in r2]


def test_captured_but_never_run_reports_nothing(tf):
    import torch

    n, batch = 256, 64
    x = torch.from_numpy(inputs.uniform(9510, batch, n, np.complex64)).cuda()
    for _ in range(2):  # the second plan may get the first one's memory
        with tf.Plan(n, batch, "c64") as plan:
            g, st = torch.cuda.CUDAGraph(), torch.cuda.Stream()
            torch.cuda.synchronize()
            out = torch.empty_like(x)
            with torch.cuda.graph(g, stream=st):
                plan.forward(x, out, stream=st)
            c, r = plan.report()
            assert c["detected"] == 0 and not r, c
            x[3, 5] = float("nan")
            plan.forward(x, ft_mode="detect")
            assert plan.report()[0]["detected"] == 1
            x[3, 5] = 1.0


# (flagged groups, one in `every` of 10000 groups of 64 signals): one gather and
# its edges, and beyond it by windows
@pytest.mark.parametrize("flagged", [1, 4095, 4096, 4097, 9999])
def test_scattered_records_come_whole_and_quickly(tf, flagged):
    import time

    import torch

    groups, n = 10000, 4
    x = torch.from_numpy(inputs.uniform(9520, 64 * groups, n, np.complex64)).cuda()
    rng = inputs.fault_rng(flagged)
    sets = {"scattered": np.sort(rng.permutation(groups)[:flagged]), "in a row": np.arange(flagged)}
    best = {}
    with tf.Plan(n, 64 * groups, "c64") as plan:
        assert plan.info()["groups"] == [groups]
        for name, hit in sets.items():
            bad = x.clone()
            bad[torch.from_numpy(64 * hit + hit % 64).cuda(), 1] = float("nan")
            plan.forward(bad, ft_mode="detect")
            c, r = plan.report()
            assert c["detected"] == c["n_records"] == flagged and c["dropped"] == 0, c
            assert [v.group for v in r] == list(hit) and all(v.action == "detected" for v in r)
            best[name] = float("inf")
            for _ in range(5):
                t0 = time.perf_counter()
                plan.report(cap=0)
                best[name] = min(best[name], time.perf_counter() - t0)
        plan.forward(x, ft_mode="detect")
        assert plan.report()[0]["detected"] == 0
    print(f"{flagged}: {best}", flush=True)
    # one copy per run of flagged groups took 20 us each
    assert best["scattered"] <= 5 * best["in a row"] + 1e-3
