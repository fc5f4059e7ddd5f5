"""GPU parity of C0 averaging, global edge keys and welding (oracle/c0.py).

Averages are summed in the same order on both sides, so they are compared
bit for bit (FP64 and FP32); keys, vertex indices and vertex counts are
integer results and also compared exactly, as are the welded vertex
coordinates (copies of the soup's own values).
"""

import numpy as np
import pytest

import workloads as W
from oracle import c0, gll, mc
from oracle import sem as osem

torch = pytest.importorskip("torch")
import paper_2312_09888_amd as sem  # noqa: E402

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def dev(a, dt=None):
    a = np.ascontiguousarray(a if dt is None else np.asarray(a, dtype=dt))
    return torch.from_numpy(a).to(DEV)


def host(t):
    return t.detach().cpu().numpy()


@pytest.mark.parametrize("dt", [np.float64, np.float32])
@pytest.mark.parametrize("shape,n", [((3, 2, 2), 4), ((4, 3, 2), 7), ((2, 2, 2), 1)])
def test_dsavg_bit_exact(dt, shape, n):
    gid = W.lattice_gid(shape, n)
    f = np.random.default_rng(n).normal(size=gid.shape).astype(dt)
    gs = sem.GatherScatter(dev(gid))
    out = sem.dsavg(dev(f), gs)
    np.testing.assert_array_equal(host(out), c0.dsavg(f, gid))
    # in place gives the same
    t = dev(f)
    sem.dsavg(t, gs, out=t)
    np.testing.assert_array_equal(host(t), c0.dsavg(f, gid))


def test_dsavg_relabelled_ids_and_unused_ids():
    shape, n = (3, 3, 2), 3
    gid = W.lattice_gid(shape, n)
    rng = np.random.default_rng(7)
    n_global = int(gid.max()) + 1
    perm = rng.permutation(n_global + 50)[:n_global]      # sparse, shuffled ids
    gid2 = perm[gid]
    f = rng.normal(size=gid.shape)
    gs = sem.GatherScatter(dev(gid2), n_global=n_global + 50)
    np.testing.assert_array_equal(host(sem.dsavg(dev(f), gs)), c0.dsavg(f, gid2))


def test_bad_ids_are_flagged():
    gid = W.lattice_gid((2, 1, 1), 2)
    gid[1, 0, 0, 0] = 10 ** 6
    st = torch.zeros(1, dtype=torch.int32, device=DEV)
    sem.GatherScatter(dev(gid), n_global=100, status=st)
    torch.cuda.synchronize()
    assert int(st.item()) & sem.SEM_FLAG_BAD_ID


def _sphere_field(shape, n, r=0.31, center=(0.5, 0.52, 0.47)):
    x, y, z = W.box_mesh(shape, n, ((0, 1.0), (0, 1.0), (0, 1.0)))
    f = r * r - ((x - center[0]) ** 2 + (y - center[1]) ** 2 + (z - center[2]) ** 2)
    return x, y, z, f


@pytest.mark.parametrize("dt", [np.float64, np.float32])
def test_global_keys_and_weld_match_oracle(dt):
    shape, n = (3, 3, 3), 5
    x, y, z, f = (a.astype(dt) for a in _sphere_field(shape, n))
    gid = W.lattice_gid(shape, n)
    t = [dev(a) for a in (x, y, z, f)]
    r = sem.isosurface(*t, [0.0], edge_keys=True)
    g = dev(gid)
    keys = sem.global_edge_keys(r["edge_key"], g)
    want = c0.global_edge_keys(host(r["edge_key"]).astype(np.uint64), gid, n)
    np.testing.assert_array_equal(host(keys).view(np.uint64), want)
    verts, idx = sem.weld(r["tri_xyz"], keys)
    ov, oi = c0.weld(host(r["tri_xyz"]), want)
    np.testing.assert_array_equal(host(idx), oi)
    np.testing.assert_array_equal(host(verts), ov)
    # the welded surface is closed across the 27 elements: V - E + F = 2
    edges = np.sort(np.concatenate([oi[:, [0, 1]], oi[:, [1, 2]], oi[:, [2, 0]]]), axis=1)
    ue, cnt = np.unique(edges, axis=0, return_counts=True)
    assert np.all(cnt == 2)
    assert ov.shape[0] - ue.shape[0] + oi.shape[0] == 2


def test_weld_overflow_and_empty():
    shape, n = (2, 2, 2), 3
    x, y, z, f = _sphere_field(shape, n, r=0.4, center=(0.5, 0.5, 0.5))
    gid = W.lattice_gid(shape, n)
    t = [dev(a) for a in (x, y, z, f)]
    r = sem.isosurface(*t, [0.0], edge_keys=True)
    keys = sem.global_edge_keys(r["edge_key"], dev(gid))
    verts, idx = sem.weld(r["tri_xyz"], keys)
    nv = verts.shape[0]
    lib = sem.lib()
    n_ref = keys.numel()
    ws = torch.empty(lib.sem_weld_workspace_bytes(n_ref), dtype=torch.uint8, device=DEV)
    small = torch.empty((nv // 2, 3), dtype=torch.float64, device=DEV)
    idx2 = torch.empty_like(idx)
    cnt = torch.zeros(1, dtype=torch.int64, device=DEV)
    st = torch.zeros(1, dtype=torch.int32, device=DEV)
    assert lib.sem_weld(n_ref, sem.SEM_F64, r["tri_xyz"].data_ptr(), keys.data_ptr(),
                        idx2.data_ptr(), small.data_ptr(), small.shape[0], cnt.data_ptr(),
                        ws.data_ptr(), ws.numel(), st.data_ptr(), None) == 0
    torch.cuda.synchronize()
    assert int(cnt.item()) == nv
    assert int(st.item()) & sem.SEM_FLAG_VERT_OVERFLOW
    assert torch.equal(idx2, idx)
    assert torch.equal(small, verts[:nv // 2])
    e = torch.empty((0, 3, 3), dtype=torch.float64, device=DEV)
    v0, i0 = sem.weld(e, torch.empty(0, dtype=torch.int64, device=DEV))
    assert v0.shape[0] == 0 and i0.shape[0] == 0


def test_averaged_q_isosurface_end_to_end():
    """Per-element Q -> C0 average -> isosurface -> weld: stage-isolated
    against the oracle on the kernel's own averaged Q, and the averaged
    field is C0 across faces."""
    shape, n = (3, 2, 2), 7
    x, y, z, u, v, w = W.tgv_config(n, shape=shape)
    gid = W.lattice_gid(shape, n)
    t = [dev(a) for a in (x, y, z, u, v, w)]
    q, _, _ = sem.qcrit(*t)
    gs = sem.GatherScatter(dev(gid))
    qa = sem.dsavg(q, gs)
    hq = host(q)
    np.testing.assert_array_equal(host(qa), c0.dsavg(hq, gid))
    oq, _, _ = osem.qcrit(x, y, z, u, v, w, gll.diff_matrix(n))
    assert np.abs(host(qa) - c0.dsavg(oq, gid)).max() < 1e-10 * np.abs(oq).max()
    c = 0.1
    r = sem.isosurface(t[0], t[1], t[2], qa, [c], edge_keys=True)
    o = mc.extract(x, y, z, host(qa), [c], edge_keys=True)
    assert int(host(r["tri_count"])[0]) == int(o["tri_count"][0])
    keys = sem.global_edge_keys(r["edge_key"], dev(gid))
    verts, idx = sem.weld(r["tri_xyz"], keys)
    okeys = c0.global_edge_keys(o["edge_key"].astype(np.uint64), gid, n)
    ov, oi = c0.weld(o["tri_xyz"], okeys)
    np.testing.assert_array_equal(host(idx), oi)
    assert np.abs(host(verts) - ov).max() <= 1e-12 * np.abs(ov).max()


@pytest.mark.parametrize("dt", [np.float64, np.float32])
@pytest.mark.parametrize("n,e,pool", [(1, 1, 3), (2, 5, 40), (3, 16, 1), (4, 700, 30000),
                                      (4, 2100, 500000)])
def test_dsavg_of_any_numbering(dt, n, e, pool):
    """Partial words, one node for all, ids without copies, nodes with bad ids
    (left alone), in place and not."""
    rng = np.random.default_rng(e)
    gid = rng.integers(0, pool, size=(e,) + (n + 1,) * 3)
    f = rng.normal(size=gid.shape).astype(dt)
    bad = rng.random(gid.shape) < 0.05
    ids = np.where(bad, rng.choice([-1, pool + 9, 1 << 40], size=gid.shape), gid)
    want = np.full_like(f, -7)
    want[~bad] = c0.dsavg(f[~bad], ids[~bad])
    st = torch.zeros(1, dtype=torch.int32, device=DEV)
    gs = sem.GatherScatter(dev(ids), n_global=pool + 9, status=st)
    out = sem.dsavg(dev(f), gs, out=torch.full_like(dev(f), -7))
    np.testing.assert_array_equal(host(out), want)
    assert bool(int(st.item()) & sem.SEM_FLAG_BAD_ID) == bool(bad.any())
    t = dev(f)
    sem.dsavg(t, gs, out=t)
    np.testing.assert_array_equal(host(t), np.where(bad, f, want))


@pytest.mark.parametrize("n_tri", [1, 682, 683, 2048, 100001])
@pytest.mark.parametrize("share", [1, 6, 500])
def test_weld_of_any_keys(n_tri, share):
    """Corners around the workgroup's number of them, from all distinct keys
    to a few that every workgroup holds; some bad keys."""
    n_ref = 3 * n_tri
    rng = np.random.default_rng(n_tri + share)
    pool = rng.integers(0, 2 ** 63, size=max(1, n_ref // share))
    keys = pool[rng.integers(0, pool.size, size=n_ref)] if share > 1 else \
        rng.permutation(n_ref).astype(np.int64) * 65536
    keys[rng.random(n_ref) < 0.01] = -1
    xyz = rng.normal(size=(n_tri, 3, 3))
    st = torch.zeros(1, dtype=torch.int32, device=DEV)
    verts, idx = sem.weld(dev(xyz), dev(keys), status=st)
    good = np.flatnonzero(keys != -1)
    _, at, inv = np.unique(keys[good], return_index=True, return_inverse=True)
    order = np.argsort(at)
    number = np.empty_like(order)
    number[order] = np.arange(order.size)
    want = np.full(n_ref, -1)
    want[good] = number[inv]
    np.testing.assert_array_equal(host(idx).ravel(), want)
    np.testing.assert_array_equal(host(verts), xyz.reshape(-1, 3)[good[at[order]]])
    assert bool(int(st.item()) & sem.SEM_FLAG_BAD_ID) == (good.size < n_ref)


def test_dsavg_takes_the_mesh_from_the_structure():
    """The structure knows its mesh: a call that names fewer elements averages
    the nodes of the set-up all the same."""
    shape, n = (3, 2, 2), 2
    e = 12
    gid = dev(W.lattice_gid(shape, n)).contiguous()
    gs = sem.GatherScatter(gid)
    f = torch.rand((e, 3, 3, 3), dtype=torch.float64, device=DEV)
    want = sem.dsavg(f, gs)
    for k in (1, 5):
        out = torch.empty_like(f)
        rc = sem.lib().sem_dsavg(k, n, sem.SEM_F64, gs.buf.data_ptr(), gs.n_global, f.data_ptr(),
                                 out.data_ptr(), torch.cuda.current_stream().cuda_stream)
        assert rc == 0 and torch.equal(out, want)


@pytest.mark.parametrize("dt", [np.float64, np.float32])
@pytest.mark.parametrize("pool", [1, 149, 160])
def test_dsavg_of_nodes_with_many_copies(dt, pool):
    """More than eight copies a node on average (and just under: 160 ids for
    1,280 nodes): lists that fit a workgroup's LDS and lists that do not."""
    rng = np.random.default_rng(pool)
    for e in (160, 1600):
        k = pool if e == 160 else 10 * pool
        gid = np.minimum(rng.integers(0, 8 * k, size=(e, 2, 2, 2)) // 8, k - 1)
        f = rng.normal(size=gid.shape).astype(dt)
        gs = sem.GatherScatter(dev(gid), n_global=k)
        t = dev(f)
        sem.dsavg(t, gs, out=t)
        np.testing.assert_array_equal(host(t), c0.dsavg(f, gid))


@pytest.mark.parametrize("n_tri", [(1 << 22) // 3, (1 << 22) // 3 + 1])
def test_weld_on_both_sides_of_four_corners_a_thread(n_tri):
    """2^22 - 1 corners (one a thread) and two more (four a thread)."""
    r = np.arange(3 * n_tri)
    keys = ((r // 7) * 2654435761) % (1 << 20)      # in runs, and again far away
    xyz = r.astype(np.float32).reshape(n_tri, 3, 1).repeat(3, axis=2)
    verts, idx = sem.weld(dev(xyz, np.float32), dev(keys))
    _, at, inv = np.unique(keys, return_index=True, return_inverse=True)
    order = np.argsort(at)
    number = np.empty_like(order)
    number[order] = np.arange(order.size)
    np.testing.assert_array_equal(host(idx).ravel(), number[inv])
    np.testing.assert_array_equal(host(verts)[:, 0], at[order].astype(np.float32))
