"""The row-group kick of small systems (fewer than 8,192 bodies) and the base
step on it, at the edges of its row groups (4), waves (64), column chunks (256)
and range, against the oracle.

Tolerances as in the parity tests: 1e-12 per acceleration of the compensated
oracle, encounter lists equal, 1e-12 of the largest component per step.
"""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_2201_10058_amd import native as N
from paper_2201_10058_amd import workload as W

pytestmark = pytest.mark.gpu

G = W.GAUSS_G
TOL = 1e-12


@pytest.mark.parametrize("dense", [False, True])
@pytest.mark.parametrize("n", [1, 2, 7, 8, 9, 64, 65, 128, 255, 257, 264, 1031, 4097, 8191])
def test_kick_and_list(dev, n, dense):
    d = W.random_cloud(n, seed=700 + n, rc_scale=0.6 if dense else 0.03)
    st = N.State.from_numpy(d)
    cfg = N.Config(G=G)
    ws = N.Workspace(n, cfg)
    oi, oj, cnt = oracle.pairs(d["x"], d["y"], d["z"], d["rc"])
    pl = N.PairList(max(cnt, 1))
    a = N.kick(st, cfg, ws, 2.0, acc=True, pairs=pl).cpu().numpy()
    assert N.read_status(ws) == N.OK
    pi, pj, c = pl.result()
    assert c == cnt and np.array_equal(pi, oi) and np.array_equal(pj, oj)
    ax, ay, az, code = oracle.kick_acc(d["x"], d["y"], d["z"], d["m"], d["rc"], G, precise=True)
    assert code == 0
    ref = np.stack([ax, ay, az])
    if n > 1:
        # a row whose every partner lies below the band has no acceleration
        size = np.linalg.norm(ref, axis=0)
        assert np.max(np.linalg.norm(a - ref, axis=0) / np.where(size > 0, size, 1.0)) <= TOL
    else:
        assert np.all(a == 0.0)
    for k, name in enumerate(("vx", "vy", "vz")):
        # v += h a in one rounding
        v = st.t[name].cpu().numpy()
        assert np.max(np.abs(v - (d[name] + 2.0 * a[k]))) <= 4e-16 * np.max(np.abs(v))


@pytest.mark.parametrize("n", [1, 2, 8, 9, 29, 64, 100, 128, 129, 200, 256, 257, 300, 2041, 5000])
def test_step_matches_oracle_and_operators(dev, n):
    spec = W.DiskSpec(f"disk_n{n}", n, 0.5, 1.5, 2.0, seed=900 + n)
    d = W.make_disk(spec)
    cfg = N.Config(G=G)
    ws = N.Workspace(n, cfg)
    st, op = N.State.from_numpy(d), N.State.from_numpy(d)
    pl, pl_op = N.PairList(64 * n), N.PairList(64 * n)
    ref = oracle.state_copy(d)
    for _ in range(3):
        assert N.step(st, cfg, ws, pl) == N.OK
        oracle.step(ref, G, 1.0, 6.0, 3.0, 0.4)
        # the same step operator by operator: the same sums in the same order,
        # except that the second kick of the step sees the positions before the
        # Sun kick that shifts them all (their differences round differently)
        N.rcrit(op, cfg, ws)
        N.kick(op, cfg, ws, 3.0, pairs=pl_op)
        N.hc(op, cfg, ws, 3.0)
        N.drift(op, cfg, ws, 6.0)
        N.hc(op, cfg, ws, 3.0)
        N.kick(op, cfg, ws, 3.0)
        assert N.read_status(ws) == N.OK
        for k in N.State.KEYS:
            assert (st.t[k] - op.t[k]).abs().max() <= 1e-15 * op.t[k].abs().max(), k
        a, b = pl.result(), pl_op.result()
        assert a[2] == b[2] and np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
    out = st.numpy()
    for k in ("x", "y", "z", "vx", "vy", "vz"):
        assert np.max(np.abs(out[k] - ref[k])) <= 3 * TOL * np.max(np.abs(ref[k])), k


def test_invalid_radius_reaches_no_column_past_the_end(dev):
    # an infinite radius is reported; the list holds real bodies only
    d = W.random_cloud(70, seed=5, rc_scale=0.1)
    rc = d["rc"].copy()
    rc[3] = np.inf
    st = N.State.from_numpy(d, rc=rc)
    cfg = N.Config(G=G)
    ws = N.Workspace(70, cfg)
    pl = N.PairList(70 * 70)
    N.kick(st, cfg, ws, 0.0, acc=True, pairs=pl)
    assert N.read_status(ws) == N.E_RCRIT
    pi, pj, c = pl.result()
    oi, oj, cnt = oracle.pairs(d["x"], d["y"], d["z"], rc)
    assert c == cnt and np.array_equal(pi, oi) and np.array_equal(pj, oj)


def test_step_graph_replay(dev):
    # captured steps against eager ones from the same state, over several replays
    d = W.make_disk(W.DiskSpec("disk_n700", 700, 0.5, 1.5, 1.0, seed=77))
    cfg = N.Config(G=G, flags=N.FLAG_NOSYNC)
    ws, ws_e = N.Workspace(700, cfg), N.Workspace(700, cfg)
    st, st_e = N.State.from_numpy(d), N.State.from_numpy(d)
    pl, pl_e = N.PairList(8192), N.PairList(8192)
    N.step(st, cfg, ws, pl)
    N.step(st_e, cfg, ws_e, pl_e)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        N.step(st, cfg, ws, pl)
    for rep in range(4):
        g.replay()
        N.step(st_e, cfg, ws_e, pl_e)
        torch.cuda.synchronize()
        for k in N.State.KEYS:
            assert torch.equal(st.t[k], st_e.t[k]), (rep, k)
        a, b = pl.result(), pl_e.result()
        assert a[2] == b[2] and np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
    assert N.read_status(ws) == N.OK and N.read_status(ws_e) == N.OK


@pytest.mark.parametrize("dense", [False, True])
@pytest.mark.parametrize("n", [1, 2, 4, 5, 64, 65, 255, 256, 257, 511, 513, 1031, 4097, 8191])
def test_kick_vjp_against_tiled_form(dev, n, dense):
    # the row-group VJP against the tiled gather form (column slices given),
    # which the autograd test pins.  Both round every term of a sum to a few
    # units of 2^-52 and add n of them in different orders, so they differ by
    # less than 64 * 2^-52 * sqrt(n) of the sum of the terms' sizes; the
    # largest gradient component stands for that sum with a factor of 64 more
    # for cancellation in it.  64 * 64 * 2^-52 * sqrt(8191) = 8e-11
    d = W.random_cloud(n, seed=40 + n, rc_scale=0.6 if dense else 0.03)
    st = N.State.from_numpy(d)
    rng = np.random.default_rng(n)
    ab = [torch.tensor(rng.normal(size=n), device="cuda") for _ in range(3)]
    base = {k: rng.normal(size=n) for k in N.AdjointState.KEYS}
    out = []
    for slices in (0, 3):
        cfg = N.Config(G=G, slices=slices)
        ws = N.Workspace(n, cfg)
        adj = N.AdjointState(n, tensors={k: torch.tensor(v, device="cuda") for k, v in base.items()})
        N.kick_vjp(st, cfg, ws, 0.7, ab, adj)
        assert N.read_status(ws) == N.OK
        out.append({k: adj.t[k].cpu().numpy() for k in adj.KEYS})
    for k in ("vx", "vy", "vz"):
        assert np.array_equal(out[0][k], base[k])
    for k in ("x", "y", "z", "m", "rc"):
        size = max(np.abs(out[1][k] - base[k]).max(), 1.0)
        assert np.abs(out[0][k] - out[1][k]).max() <= 8e-11 * size, k
    if n == 1:
        assert all(np.array_equal(out[0][k], base[k]) for k in base)
    else:
        assert np.array_equal(out[0]["rc"] != base["rc"], out[1]["rc"] != base["rc"])


def test_results_over_their_inputs(dev):
    # accelerations written over the positions and adjoints added to the arrays
    # that hold abar: as with arrays of their own (tolerances as above)
    n = 300
    d = W.random_cloud(n, seed=77, rc_scale=0.3)
    cfg = N.Config(G=G)
    ws = N.Workspace(n, cfg)
    st = N.State.from_numpy(d)
    ref = N.kick(st, cfg, ws, 0.0, acc=True).cpu().numpy()
    b, p = st.bodies(), cfg.params()
    assert N.load().genga_kick(ctypes.byref(b), ctypes.byref(p), 0.0, b.x, b.y, b.z, None, ws.ptr,
                               None) == N.OK
    torch.cuda.synchronize()
    out = np.stack([st.t[k].cpu().numpy() for k in "xyz"])
    assert np.max(np.linalg.norm(out - ref, axis=0) / np.linalg.norm(ref, axis=0)) <= TOL

    st = N.State.from_numpy(d)
    rng = np.random.default_rng(5)
    base = {k: rng.normal(size=n) for k in N.AdjointState.KEYS}
    res = []
    for shared in (False, True):
        adj = N.AdjointState(n, tensors={k: torch.tensor(v, device="cuda") for k, v in base.items()})
        ab = [adj.t[k] if shared else adj.t[k].clone() for k in "xyz"]
        N.kick_vjp(st, cfg, ws, 0.7, ab, adj)
        assert N.read_status(ws) == N.OK
        res.append({k: adj.t[k].cpu().numpy() for k in adj.KEYS})
    for k in ("x", "y", "z", "m", "rc"):
        size = max(np.abs(res[0][k] - base[k]).max(), 1.0)
        assert np.abs(res[1][k] - res[0][k]).max() <= 8e-11 * size, k


@pytest.mark.parametrize("n, k", [(200, 15), (200, 16), (300, 17), (513, 100), (2050, 40)])
def test_lists_of_rows_with_many_pairs(dev, n, k):
    # rows of up to 16 pairs go through a list, longer ones through the bitmap,
    # a wave each; on a ring of k neighbours most rows have k.  Also with a
    # capacity that ends inside a row: the list's start and the true count
    d = W.make_ring(n, neighbours=k)
    cfg = N.Config(G=G)
    ws = N.Workspace(n, cfg)
    oi, oj, cnt = oracle.pairs(d["x"], d["y"], d["z"], d["rc"], cap=n * n)
    assert cnt == n * k
    for cap in (cnt, cnt - k // 2, 0):
        st = N.State.from_numpy(d)
        pl = N.PairList(cap)
        N.kick(st, cfg, ws, 0.0, acc=True, pairs=pl)
        assert N.read_status(ws) == (N.OK if cap == cnt else N.E_OVERFLOW)
        pi, pj, c = pl.result()
        assert c == cnt and np.array_equal(pi, oi[:cap]) and np.array_equal(pj, oj[:cap])
    # in a step, where the drift's launch writes the list
    ring = W.make_bs_ring(n, neighbours=k)
    cfg = N.Config(G=ring["G"], m_star=1.0, dt=ring["dt"], n1=ring["n1"], n2=0.0)
    st = N.State.from_numpy(ring)
    pl = N.PairList(cnt)
    assert N.step(st, cfg, N.Workspace(n, cfg), pl) == N.OK
    rc = st.t["rc"].cpu().numpy()
    oi, oj, cnt = oracle.pairs(ring["x"], ring["y"], ring["z"], rc, cap=n * n)
    pi, pj, c = pl.result()
    assert c == cnt and np.array_equal(pi, oi[:cnt]) and np.array_equal(pj, oj[:cnt])


def _crowded(n, partners, seed):
    """A cloud whose bodies have about `partners` partners each, close in index
    as in space (sorted along x), so that words of 64 columns hold from none to
    all of a row's partners."""
    d = W.random_cloud(n, seed=seed)
    order = np.argsort(d["x"])
    for k in ("x", "y", "z", "m"):
        d[k] = np.ascontiguousarray(d[k][order])
    for k in ("y", "z"):
        d[k] *= 0.3 * partners / n
    d["rc"] = np.random.default_rng(seed).uniform(0.7, 1.4, n) * partners / n
    return d


CROWDED = [(129, 5), (129, 200), (300, 6), (300, 40), (2050, 4), (2050, 7), (2050, 60), (8191, 30)]


@pytest.mark.parametrize("n, partners", CROWDED)
def test_crowded_words(dev, n, partners):
    # words below and above the number of marked columns (10) from which the
    # row's wave takes them one by one, in one system
    d = _crowded(n, partners, seed=n + partners)
    oi, oj, cnt = oracle.pairs(d["x"], d["y"], d["z"], d["rc"], cap=n * n // 2 + 1)
    words = np.bincount((np.concatenate([oi, oj]).astype(np.int64) * 256 +
                         np.concatenate([oj, oi]) // 64))
    if partners < 100:
        assert words[words > 0].min() < 10
    assert words.max() >= 10
    st = N.State.from_numpy(d)
    cfg = N.Config(G=G)
    ws = N.Workspace(n, cfg)
    pl = N.PairList(cnt)
    a = N.kick(st, cfg, ws, 0.0, acc=True, pairs=pl).cpu().numpy()
    assert N.read_status(ws) == N.OK
    pi, pj, c = pl.result()
    assert c == cnt and np.array_equal(pi, oi[:cnt]) and np.array_equal(pj, oj[:cnt])
    ax, ay, az, code = oracle.kick_acc(d["x"], d["y"], d["z"], d["m"], d["rc"], G, precise=True)
    assert code == 0
    ref = np.stack([ax, ay, az])
    size = np.linalg.norm(ref, axis=0)
    assert np.max(np.linalg.norm(a - ref, axis=0) / np.where(size > 0, size, 1.0)) <= TOL


def _vjp(d, cfg, ab, base=None):
    n = d["n"]
    st = N.State.from_numpy(d)
    ws = N.Workspace(n, cfg)
    adj = N.AdjointState(n) if base is None else \
        N.AdjointState(n, tensors={k: torch.tensor(v, device="cuda") for k, v in base.items()})
    N.kick_vjp(st, cfg, ws, 0.7, ab, adj)
    assert N.read_status(ws) == N.OK
    return {k: adj.t[k].cpu().numpy() for k in adj.KEYS}


def _vjp_size(d, ab):
    """Per row and component the sum of its terms' sizes (K taken as 1 above the
    band's lower end, dK/dy as its largest value, 2)."""
    x = np.stack([d["x"], d["y"], d["z"]])
    a = 0.7 * np.stack([t.cpu().numpy() for t in ab])
    m, rc, an = d["m"], d["rc"], np.linalg.norm(a, axis=0)
    size = np.zeros((3, d["n"]))
    for i in range(d["n"]):
        r = np.linalg.norm(x - x[:, i:i + 1], axis=0)
        r[i] = 1.0
        rho = np.maximum(rc, rc[i])
        w = np.where(r > 0.1 * rho, r**-3, 0.0)
        w[i] = 0.0
        both = w * (m[i] * an + m * an[i])
        band = r < rho
        size[:, i] = ((4.0 * both).sum() + (2.5 * both * r / rho)[band].sum(), (w * r * an).sum(),
                      (2.5 * both * r**2 / rho**2)[band].sum())
    return {"x": size[0], "y": size[0], "z": size[0], "m": size[1], "rc": size[2]}


@pytest.mark.parametrize("kind", ["sparse", "dense", "crowded"])
@pytest.mark.parametrize("n", [2, 64, 65, 129, 257, 1031, 4097, 8191])
def test_kick_vjp_components_against_tiled_form(dev, n, kind):
    # each row's components against their own size, from adjoints of zero, so that no
    # base hides it.  Each term of a sum, a dozen rounded operations, is off by
    # less than 64 * 2^-52 of its size in either form, the first-order r^-5 from
    # v_rsq_f64 (e < 1.2e-7) by 35/8 e^2 < 7e-14 more, and n terms added in
    # another order by sqrt(n) * 2^-52 of the sum of the sizes
    d = _crowded(n, 6, seed=50 + n) if kind == "crowded" else \
        W.random_cloud(n, seed=50 + n, rc_scale=0.6 if kind == "dense" else 0.03)
    rng = np.random.default_rng(n)
    ab = [torch.tensor(rng.normal(size=n), device="cuda") for _ in range(3)]
    rows = _vjp(d, N.Config(G=1.0), ab)
    tiled = _vjp(d, N.Config(G=1.0, slices=3), ab)
    size = _vjp_size(d, ab)
    tol = 2 * (64 * 2.0**-52 + 7e-14) + np.sqrt(n) * 2.0**-52
    for k in ("x", "y", "z", "m", "rc"):
        assert np.all(np.abs(tiled[k]) <= 1.001 * size[k]), k
        assert np.all(np.abs(rows[k] - tiled[k]) <= tol * size[k]), k
    assert np.array_equal(rows["rc"] != 0, tiled["rc"] != 0)
    # added to what the arrays hold, in one rounding
    base = {k: rng.normal(size=n) * (np.abs(rows[k]).max() + 1e-30) for k in N.AdjointState.KEYS}
    again = _vjp(d, N.Config(G=1.0), ab, base)
    for k in N.AdjointState.KEYS:
        want = base[k] + rows[k]
        assert np.abs(again[k] - want).max() <= 2.0**-52 * (np.abs(base[k]) + np.abs(rows[k])).max(), k


def test_vjp_into_one_array_twice(dev):
    # one array for two gradients takes both sums, as in the tiled form
    n = 300
    d = W.random_cloud(n, seed=78, rc_scale=0.3)
    rng = np.random.default_rng(6)
    ab = [torch.tensor(rng.normal(size=n), device="cuda") for _ in range(3)]
    st = N.State.from_numpy(d)
    got = []
    for slices in (0, 3):
        cfg = N.Config(G=1.0, slices=slices)
        ws = N.Workspace(n, cfg)
        one = N.AdjointState(n)
        one.t["y"] = one.t["x"]
        N.kick_vjp(st, cfg, ws, 0.7, ab, one)
        assert N.read_status(ws) == N.OK
        got.append(one.t["x"].cpu().numpy())
    apart = _vjp(d, N.Config(G=1.0, slices=3), ab)
    want = apart["x"] + apart["y"]
    for g in got:
        assert np.abs(g - want).max() <= 1e-11 * np.abs(want).max()


@pytest.mark.parametrize("where", ["inside", "last"])
@pytest.mark.parametrize("n", [70, 129, 257, 300, 1031])
def test_invalid_radius_at_ragged_sizes(dev, n, where):
    # an infinite radius reaches the lanes past the last column, which repeat
    # the last body: reported, by the kick and by its VJP, and the list holds
    # real bodies only, once each
    d = W.random_cloud(n, seed=5, rc_scale=0.1)
    rc = d["rc"].copy()
    rc[3 if where == "inside" else n - 1] = np.inf
    st = N.State.from_numpy(d, rc=rc)
    cfg = N.Config(G=G)
    ws = N.Workspace(n, cfg)
    pl = N.PairList(n * n)
    N.kick(st, cfg, ws, 0.0, acc=True, pairs=pl)
    assert N.read_status(ws) == N.E_RCRIT
    pi, pj, c = pl.result()
    oi, oj, cnt = oracle.pairs(d["x"], d["y"], d["z"], rc)
    assert c == cnt and np.array_equal(pi, oi) and np.array_equal(pj, oj)
    ab = [torch.ones(n, dtype=torch.float64, device="cuda") for _ in range(3)]
    N.kick_vjp(st, cfg, ws, 1.0, ab, N.AdjointState(n))
    assert N.read_status(ws) == N.E_RCRIT


def test_largest_size_of_the_row_groups(dev):
    # 8,192 bodies take them under FLAG_DIRECTED: every word of the bitmap and
    # every sum of 256 bodies is full
    n = 8192
    cfg = N.Config(G=G, flags=N.FLAG_DIRECTED)
    d = W.random_cloud(n, seed=8, rc_scale=0.1)
    st = N.State.from_numpy(d)
    ws = N.Workspace(n, cfg)
    oi, oj, cnt = oracle.pairs(d["x"], d["y"], d["z"], d["rc"])
    pl = N.PairList(cnt)
    a = N.kick(st, cfg, ws, 0.0, acc=True, pairs=pl).cpu().numpy()
    assert N.read_status(ws) == N.OK
    pi, pj, c = pl.result()
    assert c == cnt and np.array_equal(pi, oi) and np.array_equal(pj, oj)
    ax, ay, az, code = oracle.kick_acc(d["x"], d["y"], d["z"], d["m"], d["rc"], G, precise=True)
    ref = np.stack([ax, ay, az])
    assert np.max(np.linalg.norm(a - ref, axis=0) / np.linalg.norm(ref, axis=0)) <= TOL
    rng = np.random.default_rng(n)
    ab = [torch.tensor(rng.normal(size=n), device="cuda") for _ in range(3)]
    rows = _vjp(d, N.Config(G=1.0, flags=N.FLAG_DIRECTED), ab)
    tiled = _vjp(d, N.Config(G=1.0, flags=N.FLAG_DIRECTED, slices=3), ab)
    size = _vjp_size(d, ab)
    tol = 2 * (64 * 2.0**-52 + 7e-14) + np.sqrt(n) * 2.0**-52    # (as above)
    for k in ("x", "y", "z", "m", "rc"):
        assert np.all(np.abs(rows[k] - tiled[k]) <= tol * size[k]), k
    disk = W.make_disk(W.DiskSpec("disk_n8192", n, 0.5, 2.0, 3.0, seed=91))
    st, ref = N.State.from_numpy(disk), oracle.state_copy(disk)
    pl = N.PairList(64 * n)
    for _ in range(2):
        assert N.step(st, cfg, ws, pl) == N.OK
        oracle.step(ref, G, 1.0, 6.0, 3.0, 0.4)
    out = st.numpy()
    for k in ("x", "y", "z", "vx", "vy", "vz"):
        assert np.max(np.abs(out[k] - ref[k])) <= 2 * TOL * np.max(np.abs(ref[k])), k
