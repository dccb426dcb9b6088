"""A fitting metric that is not positive definite is reported before the transform that
would divide by it: the refused call costs integrals and factorisation."""
import time

import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_refused_metric_costs_no_transform():
    """The last auxiliary shell of an alkane (730 functions, 3106 auxiliary ones) replaced by
    one that is there already: one of its pivots is zero.  The transform is most of a
    fit; half of it is left for the noise of the clock."""
    import paper_1707_03771_amd as dfx
    elems, xyz, sh, ax = W.workload("alkane")
    twin = next(s for s in reversed(ax[:-1]) if s["l"] == ax[-1]["l"])
    ws = torch.empty(dfx.eri3_plan(sh, ax)["bytes_workspace"], dtype=torch.uint8, device="cuda")
    good, refused = [], []
    for _ in range(3):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        B = dfx.eri3(sh, ax, workspace=ws)
        torch.cuda.synchronize()
        good.append(time.perf_counter() - t0)
        solve = B.info["trsm_seconds"]
        B.free()
        t0 = time.perf_counter()
        with pytest.raises(dfx.DfxError) as e:
            dfx.eri3(sh, ax[:-1] + [twin], workspace=ws)
        torch.cuda.synchronize()
        refused.append(time.perf_counter() - t0)
        assert e.value.code == dfx.ENOTPOSDEF
    print(f"fit {min(good) * 1e3:.2f} ms (transform {solve * 1e3:.2f}), refused {min(refused) * 1e3:.2f} ms")
    assert solve > 5e-3
    assert min(refused) < min(good) - 0.5 * solve
