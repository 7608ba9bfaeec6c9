"""The drift's solvers at the edges of their ranges, against the oracle: the Kepler drift on both
sides of the step at which it turns to the bracketed solver, and encounter groups of two and three
bodies at separations from the inner edge of the changeover zone to its rim; neighbour lists of a
large group with many candidate tiles."""
import numpy as np
import pytest

import discs
import oracle
import paper_2309_08217_amd as genga
from gpu_helpers import DT, System

pytestmark = pytest.mark.gpu

KEYS = ("x", "y", "z", "vx", "vy", "vz")


def _disc(r, v, m):
    st = {k: np.ascontiguousarray(a) for k, a in zip(KEYS, list(r.T) + list(v.T))}
    return discs.Disc(**st, m=m)


def _dop853(st, dt):
    """The orbits about a unit mass by a high-order integration (the oracle's solver by eccentric or
    hyperbolic anomaly does not take orbits next to the parabola)."""
    from scipy.integrate import solve_ivp
    n = len(st["x"])

    def rhs(_, y):
        r, v = y.reshape(2, 3, n)
        return np.concatenate([v.ravel(), (-r / (r * r).sum(axis=0) ** 1.5).ravel()])

    y0 = np.concatenate([st[k] for k in KEYS])
    y = solve_ivp(rhs, (0.0, dt), y0, method="DOP853", rtol=1e-13, atol=1e-15).y[:, -1]
    return dict(zip(KEYS, y.reshape(6, n)))


# from steps far below an orbit to several radians of it; |alpha| chi^2 = 1 lies near dt = 1 at 1 au
@pytest.mark.parametrize("dt", [1e-9, 1e-3, 0.3, 0.98, 1.02, 5.0])
@pytest.mark.parametrize("vfac", [(0.4, 1.0), (1.0, 1.41), (1.41, 1.43), (1.5, 3.0)])
def test_kepler_drift(dt, vfac):
    rng = np.random.default_rng(8)
    n = 200
    r, ang = rng.uniform(0.6, 2.0, n), rng.uniform(0, 2 * np.pi, n)
    f, tilt = rng.uniform(*vfac, n) / np.sqrt(r), rng.uniform(-0.3, 0.3, n)
    pos = np.stack([r * np.cos(ang), r * np.sin(ang), 0.05 * r * np.sin(3 * ang)], axis=1)
    vel = np.stack([-f * np.sin(ang + tilt), f * np.cos(ang + tilt), 0.02 * f], axis=1)
    d = _disc(pos, vel, np.zeros(n))
    s = System([d], rcrit=np.zeros(n))
    s.accel(genga.GENGA_KICK_FP64)
    genga.genga_drift(s.ctx.handle, s.b, dt)
    got = s.numpy_state()
    assert genga.genga_poll_status(s.ctx.handle) == genga.GENGA_OK
    exp = _dop853(d.state(), dt) if vfac == (1.41, 1.43) else \
        oracle.drift(d.state(), np.zeros(n), 1.0, dt, np.zeros((0, 2), np.int32))
    for k in KEYS:
        err = np.max(np.abs(got[k] - exp[k]) / np.maximum(1.0, np.abs(exp[k])))
        print(f"[kepler dt={dt} v={vfac}] {k} err {err:.2e}", flush=True)
        assert err <= 5e-12     # the bound of the drifts over many orbits
    s.close()


@pytest.mark.parametrize("members", [2, 3])
def test_groups_of_two_and_three(members):
    rng = np.random.default_rng(9)
    n, rc0 = 60, 4e-3
    r, ang = rng.uniform(0.7, 1.5, n), np.linspace(0, 2 * np.pi, n, endpoint=False)
    pos = np.stack([r * np.cos(ang), r * np.sin(ang), np.zeros(n)], axis=1)
    vel = np.stack([-np.sin(ang), np.cos(ang), np.zeros(n)], axis=1) / np.sqrt(r)[:, None]
    P, V = [pos], [vel]
    for q in range(1, members):
        u = rng.normal(size=(n, 3))
        u /= np.linalg.norm(u, axis=1)[:, None]
        P.append(pos + u * (rc0 * np.linspace(0.15, 0.95, n) / q)[:, None])
        V.append(vel + 2e-3 * rng.normal(size=(n, 3)))
    m = 10 ** rng.uniform(-11, -9, n * members)
    d = _disc(np.concatenate(P), np.concatenate(V), m)
    rc = np.where(np.arange(n * members) % 7 == 0, 1.1 * rc0, rc0)
    s = System([d], rcrit=rc)
    s.accel(genga.GENGA_KICK_FP64)
    pairs, cnt = s.encounter_list()
    assert cnt >= n
    genga.genga_drift(s.ctx.handle, s.b, DT)
    got = s.numpy_state()
    assert genga.genga_poll_status(s.ctx.handle) == genga.GENGA_OK
    exp = oracle.drift(d.state(), rc, 1.0, DT, pairs)
    for k in KEYS:
        err = np.max(np.abs(got[k] - exp[k]))
        print(f"[groups of {members}] {k} err {err:.2e}", flush=True)
        assert err <= 1e-10     # the bound of the other encounter groups
    s.close()


@pytest.mark.parametrize("tiles,last", [(31, 1), (41, 17)])
def test_one_wide_radius_in_a_long_chain(tiles, last):
    """A group along an arc, every body in reach of two neighbours on either side, and one body far
    ahead on the same orbit whose wide r_crit reaches the arc's end only: the group's largest radius
    makes most of its tiles candidates of each other (at most 32 of them, and more than 32), while
    the lists stay short."""
    n, step = 64 * tiles + last - 1, 1.5e-4
    th = np.append(np.arange(n), n - 1 + 2000) * step
    z = np.zeros(n + 1)
    pos, vel = np.stack([np.cos(th), np.sin(th), z], axis=1), np.stack([-np.sin(th), np.cos(th), z], axis=1)
    d = _disc(pos, vel, np.full(n + 1, 1e-10))
    rc = np.append(np.full(n, 2.5 * step), 2004.5 * step)
    s = System([d], rcrit=rc)
    genga.genga_set_large_groups(s.ctx.handle, True)
    s.accel(genga.GENGA_KICK_FP64)
    pairs, cnt = s.encounter_list()
    gid = oracle.groups(d.n, pairs)
    assert np.bincount(gid[gid >= 0]).max() == n + 1
    exp = oracle.drift(s.numpy_state(), rc, 1.0, DT, pairs)
    genga.genga_drift(s.ctx.handle, s.b, DT)
    got = s.numpy_state()
    assert genga.genga_poll_status(s.ctx.handle) == genga.GENGA_OK
    for k in KEYS:
        err = np.max(np.abs(got[k] - exp[k]))
        print(f"[chain of {n}] {k} err {err:.2e}", flush=True)
        assert err <= 1e-10     # the bound of the other encounter groups
    s.close()
