"""What a context does at its limits and carries (or must not carry) from one call to the next."""
import numpy as np
import pytest

import discs
import oracle
import paper_2309_08217_amd as genga
from gpu_helpers import DT, System

pytestmark = pytest.mark.gpu

FP64, FP32 = genga.GENGA_KICK_FP64, genga.GENGA_KICK_FP32
KEYS = ("x", "y", "z", "vx", "vy", "vz")


def _clusters(sizes, r_crit):
    """Clusters of the given numbers of bodies on circular orbits far from each other, members 0.8
    r_crit apart along the orbit, masses too small to matter (a pull of 2e-11 at most)."""
    c = np.arange(len(sizes))
    a0 = np.sqrt(0.25 + (16.0 - 0.25) * (c + 0.5) / len(sizes))
    ph0 = c * np.pi * (3.0 - np.sqrt(5.0))
    a = np.repeat(a0, sizes)
    ph = np.repeat(ph0, sizes) + 0.8 * r_crit / a * np.concatenate([np.arange(s) for s in sizes])
    v, zero = 1.0 / np.sqrt(a), np.zeros(len(a))
    return discs.Disc(x=a * np.cos(ph), y=a * np.sin(ph), z=zero, vx=-v * np.sin(ph), vy=v * np.cos(ph),
                      vz=zero.copy(), m=np.full(len(a), 1e-19))


# more than 8192 bodies in encounters, so that some groups lose members: as pairs alone (about 4900
# groups are left), and with groups of 12 last in the order
@pytest.mark.parametrize("sizes", [[2] * 5000, [2] * 4600 + [12] * 20])
@pytest.mark.parametrize("call", ["step", "drift"])
def test_more_bodies_in_encounters_than_the_builder_takes(sizes, call):
    """GENGA_ERR_CAPACITY, and every body moves: in its group or, left out, on its Kepler orbit.
    The masses do not matter, so both are the Kepler orbit, to the group step's 1e-12 of 4 au."""
    d = _clusters(sizes, 1e-4)
    s = System([d], rcrit=np.full(d.n, 1e-4))
    st = d.state()
    for _ in range(2):
        if call == "step":
            genga.genga_step(s.ctx.handle, s.b, DT, 1, FP64)
        else:
            _, c = s.encounter_list(standalone=True)
            assert c == sum(k - 1 for k in sizes)
            genga.genga_drift(s.ctx.handle, s.b, DT)
        assert genga.genga_poll_status(s.ctx.handle) == genga.GENGA_ERR_CAPACITY
        st = oracle.kepler_drift(st, 1.0, DT)
        got = s.numpy_state()
        err = max(np.max(np.abs(got[k] - st[k])) for k in KEYS)
        print(f"[capacity {call}] {d.n} bodies, error {err:.1e}", flush=True)
        assert err <= 1e-10
    s.close()


@pytest.mark.parametrize("levels", [1, 2])
def test_large_groups_on_a_context_with_a_history(levels):
    """A step without large groups whose list has more than 1024 pairs, other positions, large groups
    on: the next steps are those of a fresh context, bit for bit."""
    first, second = discs.disc_dense(3000, seed=5), discs.disc_dense(3000, seed=6)
    rc = oracle.rcrit(second.state(), 1.0, discs.DENSE_N1, discs.DENSE_N2, discs.DT_5_DAYS)
    assert len(oracle.encounters(first.state(), rc)) > 1024
    states = []
    for used in (True, False):
        s = System([first if used else second], rcrit=rc, pair_capacity=200000)
        h, torch = s.ctx.handle, s.torch
        if used:
            genga.genga_step(h, s.b, discs.DT_5_DAYS, 2, FP64)
            assert genga.genga_poll_status(h) == genga.GENGA_ERR_CAPACITY   # groups above 64 bodies
            for k, v in second.state().items():
                getattr(s.b, k).copy_(torch.as_tensor(v))
        genga.genga_set_large_groups(h, True)
        if levels > 1:
            rcl = torch.as_tensor(0.5 * rc, device="cuda")
            genga.genga_set_levels(h, levels, 2, rcl)
        genga.genga_step(h, s.b, discs.DT_5_DAYS, 1, FP64)
        assert genga.genga_poll_status(h) == genga.GENGA_OK, genga.genga_last_error()
        states.append(s.numpy_state())
        s.close()
    for k in KEYS:
        np.testing.assert_array_equal(states[0][k], states[1][k])


# a cluster of one tile and one of two
@pytest.mark.parametrize("size", [3, 100])
def test_coincident_bodies_under_the_levels(size):
    """Two bodies of a level's group at one place: their level kick's weight is zero, so it adds
    nothing; the Bulirsch-Stoer step of the two does not converge, is flagged and leaves them, and
    no other body sees anything of it."""
    d = _clusters([size, 2, 2], 1e-4)
    for k in KEYS:
        getattr(d, k)[1] = getattr(d, k)[0]
    s = System([d], rcrit=np.full(d.n, 1e-4))
    genga.genga_set_large_groups(s.ctx.handle, True)
    rcl = s.torch.full((d.n,), 0.5e-4, dtype=s.torch.float64, device="cuda")
    genga.genga_set_levels(s.ctx.handle, 2, 2, rcl)
    genga.genga_step(s.ctx.handle, s.b, DT, 1, FP64)
    assert genga.genga_poll_status(s.ctx.handle) == genga.GENGA_ERR_NOCONVERGE
    ref, got = oracle.kepler_drift(d.state(), 1.0, DT), s.numpy_state()
    for k in KEYS:
        assert np.all(np.isfinite(got[k]))
        assert np.max(np.abs(got[k][2:] - ref[k][2:])) <= 1e-10
    s.close()


@pytest.mark.parametrize("large", [False, True])
@pytest.mark.parametrize("steps", [1, 3])
def test_list_after_steps_is_that_of_the_positions(steps, large):
    """The list of a call's last kick is decided on the positions that the call returns: pairs whose
    r_crit is their final separation are outside, with the next number above it inside."""
    n = 800
    d = _clusters([2] * n, 1e-3)
    rng = np.random.default_rng(3)
    # approaching pairs, outside r_crit at every earlier kick and without mass, so that r_crit does not
    # change a bit of their motion; the last body's momentum gives the Sun shift
    i, j = np.arange(0, 2 * n, 2), np.arange(1, 2 * n, 2)
    for k in ("x", "y", "z"):
        u = 1e-3 * rng.normal(size=n)
        getattr(d, k)[j] = getattr(d, k)[i] + u
        getattr(d, "v" + k)[j] = getattr(d, "v" + k)[i] - 0.8 * u / (steps * DT)
    d.m[:] = 0.0
    d.m[-1] = 1e-6
    far = (np.hypot(d.x[i], d.y[i]) > 2.5) & (j < 2 * n - 1)   # little shear over the steps
    inside = rng.random(n) < 0.5
    rc = np.zeros(2 * n)
    for rim in (False, True):   # first without encounters, for the final separations
        s = System([d], rcrit=rc)
        genga.genga_set_large_groups(s.ctx.handle, large)
        genga.genga_step(s.ctx.handle, s.b, DT, steps, FP64)
        st = s.numpy_state()
        if not rim:
            dx, dy, dz = (st[k][j] - st[k][i] for k in ("x", "y", "z"))
            r2 = (dx * dx + dy * dy) + dz * dz
            lo = np.sqrt(r2)
            lo = np.where(lo * lo > r2, np.nextafter(lo, 0.0), lo)    # the largest r with r * r <= r2
            rc[i] = np.where(far, np.where(inside, np.nextafter(lo, 1.0), lo), 0.0)
        else:
            exp = oracle.encounters(st, rc)
            np.testing.assert_array_equal(exp[:, 0], i[far & inside])
            np.testing.assert_array_equal(s.encounter_list(standalone=False)[0], exp)
            np.testing.assert_array_equal(s.encounter_list(standalone=True)[0], exp)
        assert genga.genga_poll_status(s.ctx.handle) == genga.GENGA_OK, genga.genga_last_error()
        s.close()


@pytest.mark.parametrize("prec", [FP64, FP32])
def test_a_new_layout_takes_its_own_kick_plan(prec):
    """A source split set for one layout is not kept for the next: its kick is that of a fresh
    context, bit for bit."""
    d = discs.make_disc(5000, 2.5, seed=31)
    s, fresh = System([d]), System([d])
    genga.genga_set_kick_shape(s.ctx.handle, prec, 0, 3)
    assert not np.array_equal(s.accel(prec), fresh.accel(prec))   # other runs, another rounding
    genga.genga_set_systems(s.ctx.handle, s.off, s.mstar)
    np.testing.assert_array_equal(s.accel(prec), fresh.accel(prec))
    assert genga.genga_get_kick_shape(s.ctx.handle, prec) == genga.genga_get_kick_shape(fresh.ctx.handle, prec)
    s.close()
    fresh.close()


def test_no_list_after_a_refused_step():
    """genga_step refused for a group above 65536 bodies: the list of its last kick is no longer
    handed out, as after a refused genga_drift; the standalone list is."""
    n = 66000
    ph = 2.0 * np.pi * np.arange(n) / n
    zero = np.zeros(n)
    d = discs.Disc(x=np.cos(ph), y=np.sin(ph), z=zero, vx=-np.sin(ph), vy=np.cos(ph), vz=zero.copy(),
                   m=np.full(n, 1e-15))
    s = System([d], rcrit=np.full(n, 3.0 * np.pi / n))   # one neighbour on either side
    genga.genga_set_large_groups(s.ctx.handle, True)
    with pytest.raises(genga.GengaError) as e:
        genga.genga_step(s.ctx.handle, s.b, DT, 1, FP64)
    assert e.value.status == genga.GENGA_ERR_CAPACITY
    with pytest.raises(genga.GengaError) as e:
        s.encounter_list()
    assert e.value.status == genga.GENGA_ERR_STATE
    assert s.encounter_list(standalone=True)[1] == n
    s.close()


@pytest.mark.parametrize("n_sys,n", [(1, 1 << 25), (200000, 10), (200000, 65)])
def test_memory_of_a_layout(n_sys, n):
    """A layout's device memory goes by its bodies: the tasks' shares 96 B a body (four shares of
    three sums), the other arrays about 150 and some 400 a system."""
    torch = pytest.importorskip("torch")
    c = genga.Context()
    off = np.arange(n_sys + 1, dtype=np.int64) * n
    genga.genga_set_systems(c.handle, [0, 64], [1.0], 1024)   # (what a first layout leaves allocated)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    e = genga.Context()
    genga.genga_set_systems(e.handle, off, np.ones(n_sys), 1024)
    per_body = (before - torch.cuda.mem_get_info()[0]) / (n_sys * n)
    print(f"[layout] {n_sys} systems of {n}: {per_body:.0f} B a body", flush=True)
    assert per_body <= 400
    e.close()
    c.close()


# systems of every number of items (blocks of 64 bodies) that shares a workgroup with others, of none
# and of more; more of one item in a row than a workgroup has waves
SIZES = [5, 64, 65, 130, 1, 0, 512, 513, 300, 0] + [40] * 19 + [200, 3, 200, 64, 700, 7]


@pytest.mark.parametrize("call", ["step", "drift"])
def test_ensemble_of_small_systems(call):
    """Systems of their own central mass and momentum, with encounters, against the oracle."""
    ds = []
    for k, n in enumerate(SIZES):
        if n == 0:
            ds.append(discs.Disc(**{q: np.zeros(0) for q in KEYS + ("m",)}))
            continue
        d = discs.make_disc(n, 0.1 * n, seed=700 + k)
        d.mstar = 1.0 + 0.01 * k
        d.vx += 0.001 * k
        if n > 1:   # a close pair at least
            for q in KEYS:
                getattr(d, q)[n - 1] = getattr(d, q)[0] + (4e-3 if q in "xyz" else 0.0)
        ds.append(d)
    rc = [oracle.rcrit(d.state(), d.mstar, 3.0, 0.0, DT) if d.n else np.zeros(0) for d in ds]
    s = System(ds, rcrit=np.concatenate(rc))
    if call == "step":
        genga.genga_step(s.ctx.handle, s.b, DT, 3, FP64)
    else:
        s.encounter_list(standalone=True)
        genga.genga_drift(s.ctx.handle, s.b, DT)
    assert genga.genga_poll_status(s.ctx.handle) == genga.GENGA_OK, genga.genga_last_error()
    got, worst = s.numpy_state(), 0.0
    for k, d in enumerate(ds):
        if d.n == 0:
            continue
        ref = oracle.step(d.state(), rc[k], d.mstar, DT, 3)[0] if call == "step" else \
            oracle.drift(d.state(), rc[k], d.mstar, DT, oracle.encounters(d.state(), rc[k]))
        worst = max([worst] + [np.max(np.abs(got[q][s.system_slice(k)] - ref[q])) for q in KEYS])
    print(f"[ensemble {call}] {len(ds)} systems, error {worst:.1e}", flush=True)
    assert worst <= 1e-10
    s.close()


@pytest.mark.parametrize("sizes", [SIZES + [95, 96, 97, 650, 720, 2000], [800, 1100], [3]])
def test_energy_of_small_and_large_systems(sizes):
    """Runs of one length and the next, systems of less and of more than 64 tasks side by side, only
    larger ones, one alone: E and L against the oracle, to the rounding of their sums."""
    ds = [discs.make_disc(n, 2.5, seed=800 + k) if n else discs.Disc(**{q: np.zeros(0) for q in KEYS + ("m",)})
          for k, n in enumerate(sizes)]
    for k, d in enumerate(ds):
        d.mstar = 1.0 + 0.01 * k
    s = System(ds, rcrit=np.zeros(sum(sizes)))
    got = s.energy()
    for k, d in enumerate(ds):
        ref = oracle.energy(d.state(), d.mstar) if d.n else np.zeros(4)
        assert abs(got[k, 0] - ref[0]) <= 1e-13 * abs(ref[0])
        assert np.max(np.abs(got[k, 1:] - ref[1:])) <= 1e-13 * np.linalg.norm(ref[1:])
    s.close()


def test_autotune_cache_of_other_kernels(tmp_path):
    """A line without the version of the kick's kernels, as written before there was one, is not
    applied: the shapes are timed, and a line of the present version is appended."""
    d = discs.make_disc(500, 2.5, seed=41)
    s = System([d])
    path = tmp_path / "tune.txt"
    genga.genga_autotune(s.ctx.handle, s.b, FP32, str(path))
    line = path.read_text()
    words = line.split()
    assert words[:3] == ["genga-autotune", "v1", "kick2"]
    key = [w for w in words[3:-2] if w != "own"]
    path.write_text(" ".join(words[:2] + key + ["4", "1"]) + "\n")   # 4 waves, 1 share
    genga.genga_autotune(s.ctx.handle, s.b, FP32, str(path))
    lines = path.read_text().splitlines()
    assert len(lines) == 2 and lines[1].split()[:3] == words[:3]
    genga.genga_autotune(s.ctx.handle, s.b, FP32, str(path))
    assert path.read_text().splitlines() == lines
    s.close()


# 1024 rows of 16 blocks of 64 bodies are the most that every workgroup sums for itself; systems of
# one and of several workgroups beside it
@pytest.mark.parametrize("sizes", [[1 << 20], [300, (1 << 20) + 64, 2000, 30]])
def test_drift_and_step_of_a_system_of_a_million(sizes):
    """The drift against the oracle's, and a step against its own kicks and drift: four massive bodies
    a system, the others' momentum moves the Sun."""
    ds, rng = [], np.random.default_rng(9)
    for n in sizes:
        a, ph = rng.uniform(0.5, 4.0, n), rng.uniform(0.0, 2.0 * np.pi, n)
        v, zero = 1.0 / np.sqrt(a), np.zeros(n)
        ds.append(discs.Disc(x=a * np.cos(ph), y=a * np.sin(ph), z=zero, vx=0.01 - v * np.sin(ph),
                             vy=v * np.cos(ph), vz=zero.copy(), m=np.full(n, 1e-3 / n)))
    s, t = (System(ds, rcrit=np.zeros(sum(sizes))) for _ in range(2))
    for u in (s, t):
        genga.genga_set_test_bodies(u.ctx.handle, [4] * len(sizes))
    s.encounter_list(standalone=True, cap=0)
    genga.genga_drift(s.ctx.handle, s.b, DT)
    got = s.numpy_state()
    for k, d in enumerate(ds):
        ref = oracle.drift(d.state(), np.zeros(d.n), 1.0, DT, np.zeros((0, 2), np.int32))
        err = max(np.max(np.abs(got[q][s.system_slice(k)] - ref[q])) for q in KEYS)
        print(f"[million] system {k} of {d.n}, error {err:.1e}", flush=True)
        assert err <= 1e-13
    genga.genga_step(s.ctx.handle, s.b, DT, 2, FP64)
    genga.genga_drift(t.ctx.handle, t.b, DT)
    for tau in (0.5 * DT, DT):
        genga.genga_kick(t.ctx.handle, t.b, tau, FP64)
        genga.genga_drift(t.ctx.handle, t.b, DT)
    genga.genga_kick(t.ctx.handle, t.b, 0.5 * DT, FP64)
    assert all(genga.genga_poll_status(u.ctx.handle) == genga.GENGA_OK for u in (s, t))
    got, ref = s.numpy_state(), t.numpy_state()
    assert max(np.max(np.abs(got[q] - ref[q])) for q in KEYS) <= 1e-13
    s.close()
    t.close()
