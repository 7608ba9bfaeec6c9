"""The kick's task plan and candidate marks at their edges, against the FP64 oracle: source runs
of one and of several tasks, and r_crit so large that every source of a block is a candidate."""
import numpy as np
import pytest

import discs
import oracle
import paper_2309_08217_amd as genga
from gpu_helpers import System, force_errors, oracle_accel_systems

pytestmark = pytest.mark.gpu

FP64, FP32 = genga.GENGA_KICK_FP64, genga.GENGA_KICK_FP32


# 383 / 384: the last size of one run, the first of two; 33, 65: marks in the second word, a
# second block; 641: an odd last run; 4097: several chunks of masses
@pytest.mark.parametrize("n", [33, 65, 383, 384, 385, 641, 4097])
@pytest.mark.parametrize("rcrit", [0.0, 5e-3, 0.4])
def test_accel_and_list_of_the_own_plan(n, rcrit):
    d = discs.make_disc(n, 2.5, seed=500 + n, a_in=0.7, a_out=1.0)
    if n == 4097:
        d.m[1000:1003] *= 3.0   # one chunk of unequal masses among equal ones
    rc = np.full(n, rcrit)
    rc[n // 2] *= 1.5           # candidates that are no encounter pairs
    s = System([d], rcrit=rc, pair_capacity=n * n)
    ref = oracle_accel_systems(s)
    exp = oracle.encounters(d.state(), rc)
    for prec, acc, bar in ((FP64, genga.GENGA_ACC_FP64, 1e-12), (FP32, genga.GENGA_ACC_FP64, 1e-5),
                           (FP32, genga.GENGA_ACC_KAHAN32, 1e-5)):
        ax, ay, az = s.zeros(), s.zeros(), s.zeros()
        genga.genga_accel(s.ctx.handle, s.b, ax, ay, az, prec, acc)
        s.torch.cuda.synchronize()
        a = np.stack([v.cpu().numpy() for v in (ax, ay, az)], axis=1)
        rms, mx = force_errors(a, ref)
        print(f"[own plan] n={n} rcrit={rcrit} prec={prec} acc={acc} rms={rms:.2e} max={mx:.2e}", flush=True)
        assert rms <= bar
        np.testing.assert_array_equal(s.encounter_list(cap=n * n)[0], exp)
    np.testing.assert_array_equal(s.encounter_list(cap=n * n, standalone=True)[0], exp)
    assert genga.genga_poll_status(s.ctx.handle) == genga.GENGA_OK
    s.close()


@pytest.mark.parametrize("n,wide", [(600, 0), (700, 0), (2500, 0), (3000, 300), (8000, 7999)])
def test_long_lists_in_order(n, wide):
    """Lists on both sides of the length that one workgroup sorts (512 pairs), with a body in the
    middle of the order that has few partners, more than are ranked by counting (256) and more than
    fit LDS (6144): the oracle's list, pair for pair."""
    d = discs.disc_dense(n, seed=11)
    rc = oracle.rcrit(d.state(), d.mstar, discs.DENSE_N1, discs.DENSE_N2, discs.DT_5_DAYS)
    if wide:
        st = d.state()
        r = np.sort(np.sqrt(sum((st[k] - st[k][n // 2 if wide < n - 1 else 0]) ** 2 for k in ("x", "y", "z"))))
        rc[n // 2 if wide < n - 1 else 0] = 2.0 * r[-1] if wide >= n - 1 else 0.5 * (r[2 * wide] + r[2 * wide + 1])
    exp = oracle.encounters(d.state(), rc)
    s = System([d], pair_capacity=len(exp) + 64, rcrit=rc)
    got, cnt = s.encounter_list(cap=len(exp) + 64, standalone=True)
    print(f"[list n={n}] {cnt} pairs, most of a body {np.bincount(exp[:, 0]).max()}", flush=True)
    assert cnt == len(exp) and (cnt > 512) == (n > 600) and (cnt > 1024) == (n > 700)
    if wide:
        assert np.bincount(exp[:, 0]).max() > (256 if wide < n - 1 else 6144)
    np.testing.assert_array_equal(got, exp)
    s.close()


@pytest.mark.parametrize("sizes", [[7647], [7648], [1535] * 40, [1537] * 40, [600, 7700, 1, 130]])
def test_accel_on_both_sides_of_the_longer_runs(sizes):
    """The first size of one disc whose runs are of 512 sources and the one before it; discs just
    too small for them although there are tasks enough, and just large enough; uneven ones."""
    ds = [discs.make_disc(n, 2.5, seed=900 + k, a_in=0.7, a_out=1.0) for k, n in enumerate(sizes)]
    s = System(ds)
    ref = oracle_accel_systems(s)
    for prec, bar in ((FP64, 1e-12), (FP32, 1e-5)):
        ax, ay, az = s.zeros(), s.zeros(), s.zeros()
        genga.genga_accel(s.ctx.handle, s.b, ax, ay, az, prec, genga.GENGA_ACC_FP64)
        s.torch.cuda.synchronize()
        a = np.stack([v.cpu().numpy() for v in (ax, ay, az)], axis=1)
        rms, mx = force_errors(a, ref)
        print(f"[runs] sizes={sizes[:4]} prec={prec} rms={rms:.2e} max={mx:.2e}", flush=True)
        assert rms <= bar
    assert genga.genga_poll_status(s.ctx.handle) == genga.GENGA_OK
    s.close()
