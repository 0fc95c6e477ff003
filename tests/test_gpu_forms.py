"""Launch forms where they begin and end: tile launches of three passes (a middle
strided pass) and on both sides of their limit; turn kernels in place and on
ragged classes, whose signals lie where an offset table says.  Every case
asserts the form that runs."""
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


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n,batch,passes,form", [(1 << 15, 1, 3, "tile"), (1 << 15, 2, 3, "tile"), (1 << 16, 3, 3, "tile"),
                                                 (1 << 18, 1, 3, "tile"), (512, 16384, 0, "tile"), (512, 16448, 0, "turns")])
def test_tiles_of_three_passes_and_at_the_limit(tf, dtype, n, batch, passes, form):
    import torch

    assert set(tf.forms(n, batch, dtype, passes=passes)) == {form}
    rng = inputs.fault_rng(n + batch)
    x = inputs.uniform(9600 + batch % 89, batch, n, NPDT[dtype])
    xd = torch.from_numpy(x).cuda()
    rows = sorted({0, batch // 2, batch - 1})
    want = {inv: oracle.fft(x[rows].astype(np.complex128), inverse=inv) for inv in (False, True)}
    print(f"forms {dtype} {n} x {batch} passes={passes}", flush=True)
    with tf.Plan(n, batch, dtype, passes=passes) as plan, tf.Plan(n, batch, dtype, passes=passes, grid_scale=1) as ref:
        info = plan.info()
        for p in range(info["passes"]):
            done = math.prod(info["pass_len"][: p + 1])
            sig, idx = int(rng.integers(batch)), int(rng.integers(n))
            # 64 x the RMS: far above the rounding noise of the group's checksum
            fault = [dict(signal=sig, pass_=p, stage=int(rng.integers(info["stages"][p])), index=idx,
                          value=64.0 * math.sqrt(2.0 * done / 3.0) * (0.6 - 0.8j))]
            for mode, inverse, faults in [("off", True, []), ("detect", False, fault), ("correct", True, fault),
                                          ("correct", False, [])]:
                got = []
                for q in (plan, ref):
                    q.set_faults(faults)
                    y = (q.inverse if inverse else q.forward)(xd, ft_mode=mode)
                    got.append((y.cpu().numpy(), *q.report()))
                (y, c, r), (yr, cr, rr) = got
                assert c == cr and c["detected"] == len(faults) and c["uncorrectable"] == 0, (p, mode, c, cr)
                assert [(a.signal, a.sub, a.group, a.pass_, a.member, a.action, a.method) for a in r] == [
                    (a.signal, a.sub, a.group, a.pass_, a.member, a.action, a.method) for a in rr]
                assert all((a.signal, a.pass_, a.sub) == (sig, p, idx // info["pass_len"][p] if info["passes"] > 1 else 0)
                           for a in r)
                if mode == "detect":
                    continue
                assert oracle.rel_l2(y[rows], want[inverse]) <= TOL[dtype]
                assert oracle.rel_l2(y, yr) <= TOL[dtype]


# groups shared by workgroups, with a partial last one; whole groups begun apart
TURNS = [("c64", 4096, 1041), ("c64", 4096, 4111), ("c64", 1024, 4161), ("c128", 1024, 12353), ("c128", 512, 16449)]


@pytest.mark.parametrize("dtype,n,batch", TURNS)
def test_turns_in_place(tf, dtype, n, batch):
    import torch

    assert tf.forms(n, batch, dtype) == ["turns"]
    x = inputs.uniform(9650 + n % 83, batch, n, NPDT[dtype])
    xd = torch.from_numpy(x).cuda()
    rows = sorted({0, 1, batch // 2, batch - 2, batch - 1})
    print(f"in place {dtype} {n} x {batch}", flush=True)
    with tf.Plan(n, batch, dtype) as plan:
        for mode in ("off", "detect"):
            for inverse in (False, True):
                fn = plan.inverse if inverse else plan.forward
                y = fn(xd, ft_mode=mode)
                z = xd.clone()
                fn(z, out=z, ft_mode=mode)
                assert bool((z == y).all()) and plan.report()[0]["detected"] == 0
                ref = oracle.fft(x[rows].astype(np.complex128), inverse=inverse)
                assert oracle.rel_l2(z[rows].cpu().numpy(), ref) <= TOL[dtype]


@pytest.mark.parametrize("dtype,n,count", TURNS)
def test_turns_ragged_offsets(tf, dtype, n, count):
    """One length class whose signals lie in reverse order with gaps."""
    import torch

    assert tf.forms(n, count, dtype) == ["turns"]
    off = (np.arange(count, dtype=np.int64)[::-1] * (n + 6)).copy()
    total = int(off.max()) + n
    x = inputs.uniform_flat(9700 + n % 79, total, NPDT[dtype])
    print(f"ragged rows {dtype} {n} x {count}", flush=True)
    rg = tf.Ragged(np.full(count, n, np.int64), off, dtype)
    hit = [0, count // 2, count - 1]
    rg.set_faults([dict(signal=s, pass_=0, stage=0, index=(7 * s + 5) % n, value=64.0 * math.sqrt(2.0 * n / 3.0)) for s in hit])
    xd = torch.from_numpy(x).cuda()
    out = torch.full_like(xd, 7 + 7j)
    rg.forward(xd, out)
    c, r = rg.report()
    y = out.cpu().numpy()
    assert c["corrected"] == len(hit) and sorted(q.signal for q in r) == hit, (c, r)
    covered = np.zeros(total, bool)
    for i in range(count):
        covered[off[i]:off[i] + n] = True
    assert np.all(y[~covered] == 7 + 7j)
    for i in sorted({*hit, 1, count - 2}):
        assert oracle.rel_l2(y[off[i]:off[i] + n], oracle.fft(x[off[i]:off[i] + n].astype(np.complex128)[None])[0]) <= TOL[dtype], i
