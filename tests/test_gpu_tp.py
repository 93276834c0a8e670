"""Test-particle modes 1 and 2 (Sect. 8) of the binary64 kick, pair list and
step against the oracle's test-particle functions (pinned in test_oracle_tp.py).
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
ACC_TOL = 1e-12


def _say(*a):
    print(*a, flush=True)


def _cloud(n, nm, seed, rc_scale=0.3):
    d = dict(W.random_cloud(n, seed=seed, rc_scale=rc_scale))
    m = d["m"].copy()
    m[:nm] *= 50.0
    d["m"] = m
    return d


def _kick(d, rc, nm, mode, ipt=0):
    st = N.State.from_numpy(d, rc=rc)
    cfg = N.Config(G=G, tp_mode=mode, n_massive=nm, ipt=ipt)
    ws = N.Workspace(st.n, cfg)
    cap = max(16, oracle.pairs_tp(d["x"], d["y"], d["z"], rc, nm, mode, cap=0)[2])
    pl = N.PairList(cap)
    a = N.kick(st, cfg, ws, 0.0, acc=True, pairs=pl)
    torch.cuda.synchronize()
    return a.cpu().numpy(), pl.result(), N.read_status(ws)


def _check(d, rc, nm, mode, ipt=0):
    a, (pi, pj, cnt), code = _kick(d, rc, nm, mode, ipt)
    assert code == N.OK
    ax, ay, az, st = oracle.kick_acc_tp(d["x"], d["y"], d["z"], d["m"], rc, G, nm, mode, precise=True)
    ref = np.stack([ax, ay, az])
    scale = np.linalg.norm(ref, axis=0)
    nz = scale > 0
    err = np.zeros(ref.shape[1])
    err[nz] = np.linalg.norm(a - ref, axis=0)[nz] / scale[nz]
    assert np.all(a[:, ~nz] == 0.0)
    opi, opj, ocnt = oracle.pairs_tp(d["x"], d["y"], d["z"], rc, nm, mode)
    _say(f"tp{mode} n={rc.size} nm={nm}: max rel err {err.max():.3e}, pairs {cnt}")
    assert err.max() <= ACC_TOL
    assert cnt == ocnt and np.array_equal(pi, opi) and np.array_equal(pj, opj)


@pytest.mark.parametrize("mode", [1, 2])
@pytest.mark.parametrize("n,nm,ipt", [(600, 37, 1), (257, 256, 2), (1000, 1, 1), (300, 300, 1)])
def test_tp_kick_random(dev, mode, n, nm, ipt):
    d = _cloud(n, nm, seed=n + nm)
    _check(d, d["rc"], nm, mode, ipt)


@pytest.mark.parametrize("mode", [1, 2])
def test_tp_kick_disk(dev, mode):
    d = W.make_tp_disk(4096, 16, seed=31)
    rc = oracle.rcrit(d["x"], d["y"], d["z"], d["vx"], d["vy"], d["vz"], d["m"], 1.0, 6.0, 3.0, 0.4)
    _check(d, rc, 16, mode)


@pytest.mark.parametrize("mode", [1, 2])
def test_tp_kick_disk65536_sampled(dev, mode):
    # the benchmark's test-particle disk (16 massive bodies, 65,520 test
    # particles) in the launch configuration the benchmark times: every
    # massive row (1,024 column slices each) and two blocks of test-particle
    # rows against the oracle, and the whole encounter list
    d = W.make_tp_disk(65536, 16)
    rc = oracle.rcrit(d["x"], d["y"], d["z"], d["vx"], d["vy"], d["vz"], d["m"], 1.0, 6.0, 3.0, 0.4)
    a, (pi, pj, cnt), code = _kick(d, rc, 16, mode)
    assert code == N.OK
    for i0, i1 in ((0, 16), (16, 2064), (63488, 65536)):
        ax, ay, az, st = oracle.kick_acc_tp(d["x"], d["y"], d["z"], d["m"], rc, G, 16, mode,
                                            rows=(i0, i1), precise=True)
        assert st == 0
        ref = np.stack([ax, ay, az])
        err = np.linalg.norm(a[:, i0:i1] - ref, axis=0) / np.linalg.norm(ref, axis=0)
        _say(f"tp{mode} disk65536 rows [{i0}, {i1}): max rel err {err.max():.3e}")
        assert err.max() <= ACC_TOL
    opi, opj, ocnt = oracle.pairs_tp(d["x"], d["y"], d["z"], rc, 16, mode)
    _say(f"tp{mode} disk65536 pairs {cnt}")
    assert cnt == ocnt and np.array_equal(pi, opi) and np.array_equal(pj, opj)


@pytest.mark.parametrize("mode", [1, 2])
def test_tp_no_massive_body(dev, mode):
    d = _cloud(500, 0, seed=77)
    a, (pi, pj, cnt), code = _kick(d, d["rc"], 0, mode)
    assert code == N.OK and cnt == 0
    assert not np.any(a)


@pytest.mark.parametrize("mode", [1, 2])
def test_tp_step_matches_oracle(dev, mode):
    d = W.make_tp_disk(2048, 16, seed=32)
    st = N.State.from_numpy(d)
    cfg = N.Config(G=G, tp_mode=mode, n_massive=16)
    ws = N.Workspace(st.n, cfg)
    ref = oracle.state_copy(d)
    pl = N.PairList(1 << 16)
    for _ in range(10):
        x0 = {c: st.t[c].cpu().numpy().copy() for c in "xyz"}
        assert N.step(st, cfg, ws, pl) == N.OK
        pi, pj, cnt = pl.result()
        rc = st.t["rc"].cpu().numpy()
        opi, opj, ocnt = oracle.pairs_tp(x0["x"], x0["y"], x0["z"], rc, 16, mode)
        assert cnt == ocnt and np.array_equal(pi, opi) and np.array_equal(pj, opj)
        oracle.step_tp(ref, G, 1.0, 6.0, 3.0, 0.4, 16, mode)
    out = st.numpy()
    for keys in (("x", "y", "z"), ("vx", "vy", "vz")):
        g = np.stack([out[k] for k in keys])
        r = np.stack([ref[k] for k in keys])
        e = np.max(np.abs(g - r)) / np.max(np.abs(r))
        _say(f"tp{mode} 10 steps {keys[0]}: {e:.3e}")
        assert e < 1e-12


def test_tp_unsupported_combinations(dev):
    d = _cloud(300, 10, seed=5)
    st = N.State.from_numpy(d, rc=d["rc"])
    cfg = N.Config(G=G, tp_mode=2, n_massive=10, precision=N.MIXED)
    ws = N.Workspace(st.n, cfg)
    with pytest.raises(N.GengaError) as e:
        N.kick(st, cfg, ws, 0.0)
    assert e.value.code == N.E_UNSUPPORTED
    cfg = N.Config(G=G, tp_mode=2, n_massive=10)
    with pytest.raises(N.GengaError) as e:
        N.energy(st, cfg, ws)
    assert e.value.code == N.E_UNSUPPORTED
    cfg = N.Config(G=G, tp_mode=1, n_massive=301)
    with pytest.raises(N.GengaError) as e:
        N.kick(st, cfg, ws, 0.0)
    assert e.value.code == N.E_INVAL


# the kick that evaluates a pair once for both bodies (1 to 64 massive bodies)
# and its neighbour above: sizes around its blocks (256), waves (64) and groups
# of 4 massive bodies, sparse and with every pair inside its radius
@pytest.mark.parametrize("mode", [1, 2])
@pytest.mark.parametrize("dense", [False, True])
@pytest.mark.parametrize("n,nm", [(2, 1), (65, 64), (256, 4), (257, 5), (300, 63), (513, 64),
                                  (600, 65), (4100, 17)])
def test_tp_kick_edges(dev, mode, dense, n, nm):
    d = _cloud(n, nm, seed=3 * n + nm)
    _check(d, d["rc"] * (8.0 if dense else 0.2), nm, mode)


@pytest.mark.parametrize("mode", [1, 2])
@pytest.mark.parametrize("n,nm", [(2, 1), (257, 3), (700, 64), (700, 65)])
def test_tp_step_matches_operators(dev, mode, n, nm):
    # the fused step against its operators one by one: the same sums, except
    # that its second kick sees the positions before their common shift
    d = W.make_tp_disk(n, nm, seed=33)
    cfg = N.Config(G=G, tp_mode=mode, n_massive=nm)
    ws = N.Workspace(n, cfg)
    st, op = N.State.from_numpy(d), N.State.from_numpy(d)
    pl, pl_op = N.PairList(64 * n), N.PairList(64 * n)
    ref = oracle.state_copy(d)
    for _ in range(3):
        assert N.step(st, cfg, ws, pl) == N.OK
        oracle.step_tp(ref, G, 1.0, 6.0, 3.0, 0.4, nm, mode)
        N.rcrit(op, cfg, ws)
        N.kick(op, cfg, ws, 3.0, pairs=pl_op)
        N.hc(op, cfg, ws, 3.0)
        N.drift(op, cfg, ws, 6.0)
        N.hc(op, cfg, ws, 3.0)
        N.kick(op, cfg, ws, 3.0)
        assert N.read_status(ws) == N.OK
        a, b = pl.result(), pl_op.result()
        assert a[2] == b[2] and np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
    out = st.numpy()
    for k in ("x", "y", "vx", "vy", "rc"):
        assert (st.t[k] - op.t[k]).abs().max() <= 1e-14 * op.t[k].abs().max(), k
    for k in ("x", "y", "z", "vx", "vy", "vz"):
        assert np.max(np.abs(out[k] - ref[k])) <= 3e-12 * max(np.max(np.abs(ref[k])), 1e-3), k


def test_tp_graph_replay(dev):
    d = W.make_tp_disk(3000, 16, seed=34)
    cfg = N.Config(G=G, tp_mode=2, n_massive=16, flags=N.FLAG_NOSYNC)
    ws, ws_e = N.Workspace(3000, cfg), N.Workspace(3000, cfg)
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


@pytest.mark.parametrize("mode", [1, 2])
def test_tp_results_over_their_inputs(dev, mode):
    # accelerations written over the positions: as with arrays of their own
    # (both within the oracle's bound of the accelerations)
    n, nm = 700, 9
    d = _cloud(n, nm, seed=41)
    cfg = N.Config(G=G, tp_mode=mode, n_massive=nm)
    ws = N.Workspace(n, cfg)
    st = N.State.from_numpy(d)
    ref = N.kick(st, cfg, ws, 0.0, acc=True).cpu().numpy()
    b, p = st.bodies(), cfg.params()
    assert N.load().genga_kick(ctypes.byref(b), ctypes.byref(p), 0.0, b.x, b.y, b.z, None, ws.ptr,
                               None) == N.OK
    assert N.read_status(ws) == N.OK
    out = np.stack([st.t[k].cpu().numpy() for k in "xyz"])
    size = np.linalg.norm(ref, axis=0)
    assert np.max(np.linalg.norm(out - ref, axis=0) / np.where(size > 0, size, 1.0)) <= 2 * ACC_TOL
