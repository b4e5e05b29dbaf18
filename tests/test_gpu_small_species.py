"""Kernels chosen for small species against the general ones: the same particles
in a species whose capacity takes either side of the rule give the same photons
and pairs.  The two compile the same device functions, so ids, counts and order
are equal and values agree to a few roundings of their type (an event's dozen
float32 or float64 operations in a row: 64 units in the last place)."""
import math

import numpy as np
import pytest

from tests.gpu_helpers import need_gpu

import workloads

pytestmark = pytest.mark.gpu

SMALL, LARGE = 1 << 17, (1 << 17) + 1              # capacities either side of the emission's rule
PAIR_SMALL, PAIR_LARGE = 1 << 18, (1 << 18) + 1    # and of the float64 pair pass's
ULPS = {"f32": 64 * 2.0 ** -24, "f64": 64 * 2.0 ** -53}


def _same(a, b, dtype):
    assert np.array_equal(a["id"], b["id"])
    for k in ("x", "p"):
        scale = np.maximum(np.abs(b[k]), np.abs(b[k]).max(axis=1, keepdims=True)) if b[k].size else b[k]
        assert np.all(np.abs(a[k] - b[k]) <= ULPS[dtype] * scale)
    # the optical depth: a float64 draw, less a rate of the species' precision
    assert np.all(np.abs(a["tau"] - b["tau"]) <= ULPS[dtype] * np.maximum(1.0, np.abs(b["tau"])))


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("method1", [False, True])
@pytest.mark.parametrize("n,dt", [(0, 0.01), (1, 2.0), (255, 2.0), (256, 0.01), (257, 2.0), (5000, 0.01), (5000, 2.0),
                                  (SMALL, 0.02)])
def test_emission_small_equals_list(dtype, method1, n, dt):
    """dt = 2: nearly every electron emits, so tiles are full and the cap is
    reached; 0.01: a few emitters per tile."""
    torch, q = need_gpu()
    ens = workloads.uniform_b_ensembles(max(n, 1), seed=5, triples=((2000.0, 206.0),))[0]
    out = []
    for cap in (SMALL, LARGE):
        ctx = q.Context(seed=9, kmax=4, flags=q.QED_FLAG_METHOD_I if method1 else 0)
        ctx.qed_build_tables(q.QED_FORMULA_I)
        lep, ph = q.Species(cap, dtype), q.Species(12 * max(n, 1), dtype)
        lep.load(ens["x"][:n], ens["p"][:n], np.zeros(n), ens["id"][:n])
        ctx.qed_init_optical_depth(lep, 0)
        ctx.qed_set_next_id(n)
        fld = q.Fields(q.QED_FIELD_UNIFORM, B=(0, 0, 2000.0))
        print(f"emission: {dtype} method1={method1} n={n} dt={dt} capacity {cap}", flush=True)
        for s in range(3):
            ctx.qed_gather_push(fld, lep, -1, dt, s)
            ctx.qed_emit_photons(lep, ph, s)
        st, _ = ctx.qed_get_status()
        out.append((lep.to_numpy(), ph.to_numpy(), st))
        ctx.close()
    (la, pa, sa), (lb, pb, sb) = out
    assert sa == sb
    assert sa["photons"] == pa["id"].size and (n < 200 or sa["photons"] > 0)
    _same(la, lb, dtype)
    _same(pa, pb, dtype)


@pytest.mark.parametrize("n", [0, 1, 255, 257, 20000, PAIR_SMALL])
def test_pairs_f64_one_and_four_photons_per_thread(n):
    torch, q = need_gpu()
    w = workloads.pair_photons(max(n, 1), seed=6, chi_lo=1.0)
    perp = np.linalg.norm(np.cross(w["khat"], w["E"] + np.cross(w["khat"], w["B"])), axis=1)
    k = w["khat"] * (w["chi_target"] * (510998.95 / 1.239841984) / perp)[:, None]
    out = []
    for cap in (PAIR_SMALL, PAIR_LARGE):
        ctx = q.Context(seed=2, kmax=4, flags=q.QED_FLAG_TRACK_DEAD)
        ctx.qed_build_tables(q.QED_FORMULA_I)
        ph, el, po = q.Species(cap, "f64"), q.Species(max(n, 1), "f64"), q.Species(max(n, 1), "f64")
        ph.load(w["x"][:n], k[:n], np.zeros(n), w["id"][:n])
        e0 = np.zeros((0, 3))
        for sp in (el, po):
            sp.load(e0, e0, np.zeros(0), np.zeros(0, np.uint64))
        ctx.qed_init_optical_depth(ph, 0)
        ctx.qed_set_next_id(n)
        fld = q.Fields(q.QED_FIELD_UNIFORM, E=(100.0, -50.0, 30.0), B=(0, 0, 2000.0))
        print(f"pairs f64: n={n} capacity {cap}", flush=True)
        for s in range(3):
            ctx.qed_create_pairs(fld, ph, el, po, 0.02, s)
            ctx.qed_compact(ph)
        st, _ = ctx.qed_get_status()
        out.append(([sp.to_numpy() for sp in (ph, el, po)], st))
        ctx.close()
    (a, sa), (b, sb) = out
    assert sa == sb
    assert sa["pairs"] == a[1]["id"].size and (n < 1000 or sa["pairs"] > 0)
    for x, y in zip(a, b):
        _same(x, y, "f64")


@pytest.mark.parametrize("order", ["sorted", "random"])
@pytest.mark.parametrize("n", [600_001, 513])
def test_wide_workgroups_of_a_sparse_species(order, n):
    """The 512-thread lepton pass (fewer than five particles per cell, capacity of
    at least 2^19) against the 256-thread one (a larger capacity): the same
    emitters and photons, values to float32 rounding (positions within 2 units in
    the last place of the box length, momenta within 16 of the larger of |p| and
    the kick a0 dt, optical depths within the rate's 1e-6), from staged boxes
    and from the global gather."""
    torch, q = need_gpu()
    ng, L, dt, a0 = 64, workloads.BOX_L, 0.01, 500.0
    ens = workloads.standing_wave_electrons(n, seed=8)
    tau = np.random.default_rng(1).exponential(size=n)
    grid = torch.empty(ng ** 3 * 6, dtype=torch.float32, device="cuda")
    fld = q.Fields(q.QED_FIELD_GRID, grid=grid, n=ng, L=L)
    out = []
    for cap in (600_001, 5 * ng ** 3):
        print(f"sparse lepton pass: n={n} {order} capacity {cap}", flush=True)
        ctx = q.Context(seed=3, kmax=4)
        ctx.qed_build_tables(q.QED_FORMULA_I)
        ctx.qed_fill_standing_wave(grid, ng, L, a0, 0.21)
        src, lep, ph = q.Species(cap, "f32"), q.Species(cap, "f32"), q.Species(200_000, "f32")
        src.load(ens["x"], ens["p"], tau, ens["id"])
        if order == "sorted":
            ctx.qed_sort_by_cell(fld, src, lep)
        else:
            lep = src
        ctx.qed_set_next_id(n)
        ctx.qed_gather_push(fld, lep, -1, dt, 0)
        ctx.qed_emit_photons(lep, ph, 0)
        st, _ = ctx.qed_get_status()
        out.append((lep.to_numpy(), ph.to_numpy(), st))
        ctx.close()
    (a, pa, sa), (b, pb, sb) = out
    assert sa["events"] == sb["events"] > 0
    if n > 1000:            # (tiles that straddle two distant blocks fall back in cell order too)
        tiles = -(-n // 512)
        assert sa["box_fallback"] == tiles if order == "random" else sa["box_fallback"] < tiles // 2
    assert np.array_equal(a["id"], b["id"]) and np.array_equal(pa["id"], pb["id"])
    assert np.max(np.abs(a["x"] - b["x"])) <= 2.0 ** -20
    assert np.max(np.abs(a["p"] - b["p"]) / np.maximum(np.abs(b["p"]), a0 * dt)) <= 2.0 ** -19
    np.testing.assert_allclose(a["tau"], b["tau"], rtol=1e-6, atol=1e-6)
    np.testing.assert_allclose(pa["p"], pb["p"], rtol=1e-5, atol=1e-4)


@pytest.mark.parametrize("surrogate", [False, True])
@pytest.mark.parametrize("n", [1, 255, 257, 300_001])
def test_photon_pass_on_a_grid_staged_equals_global(n, surrogate):
    """Photons in cell order stage their stencil boxes in LDS, the same photons in
    random order gather from global memory: optical depths, positions and the
    converted ones, matched by id, are the same bit for bit (one kernel, one
    arithmetic), every third photon dead and in place."""
    torch, q = need_gpu()
    ng, L, dt = 32, workloads.BOX_L, 0.01
    rng = np.random.default_rng(n)
    x = rng.uniform(0.0, L, (n, 3))
    k = rng.normal(size=(n, 3))
    k *= (10.0 ** rng.uniform(0.0, 4.0, n) / np.linalg.norm(k, axis=1))[:, None]
    tau = rng.exponential(size=n) * 0.05
    ids = np.arange(n, dtype=np.uint64)
    ids[1::3] = np.uint64(0xFFFFFFFFFFFFFFFF)
    cell = np.floor(x / (L / ng) + 0.5).astype(np.int64) % ng
    blk = cell // 4
    order = np.lexsort((cell[:, 0], cell[:, 1], cell[:, 2], blk[:, 0], blk[:, 1], blk[:, 2]))
    res = []
    for perm in (order, rng.permutation(n)):
        ctx = q.Context(seed=3, kmax=4, flags=q.QED_FLAG_SURROGATE if surrogate else 0)
        ctx.qed_build_tables(q.QED_FORMULA_I)
        if surrogate:                       # (weights of any kind: a rate outside the envelope takes the table)
            for net in (0, 1):
                m = q.lib().qed_surrogate_params(net)
                ctx.qed_surrogate_io(net, np.random.default_rng(net).normal(0, 0.05, m).astype(np.float32))
        grid = torch.empty(ng ** 3 * 6, dtype=torch.float32, device="cuda")
        fld = q.Fields(q.QED_FIELD_GRID, grid=grid, n=ng, L=L)
        ctx.qed_fill_standing_wave(grid, ng, L, 1000.0, 0.3)
        ph, el, po = q.Species(n + 7, "f32"), q.Species(n + 1, "f32"), q.Species(n + 1, "f32")
        ph.load(x[perm], k[perm], tau[perm], ids[perm])
        e0 = np.zeros((0, 3))
        for sp in (el, po):
            sp.load(e0, e0, np.zeros(0), np.zeros(0, np.uint64))
        ctx.qed_set_next_id(n)
        print(f"photon pass on a grid: n={n} surrogate={surrogate}", flush=True)
        ctx.qed_create_pairs(fld, ph, el, po, dt, 0)
        st, _ = ctx.qed_get_status()
        g = ph.to_numpy()
        back = np.argsort(perm)
        res.append((g["tau"][back], g["x"][back], g["id"][back], st["pairs"], st["nan_chi"]))
        ctx.close()
    a, b = res
    assert a[3:] == b[3:] and (n < 1000 or a[3] > 0)
    for u, v in zip(a[:3], b[:3]):
        assert np.array_equal(u, v)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("n", [0, 1, 3, 4, 1023, 1024, 1029, 8193])
def test_sort_moves_every_array(dtype, n):
    """All arrays of a species go through one permutation at the ends of its groups of
    four and of its blocks; the values are moved, so they are equal bit for bit."""
    torch, q = need_gpu()
    rng = np.random.default_rng(n + 1)
    ng, L = 12, 2 * math.pi
    x = rng.uniform(0, L, (n, 3)).astype(np.float32).astype(np.float64)
    p = rng.normal(size=(n, 3)).astype(np.float32).astype(np.float64)
    tau, ids = rng.uniform(size=n), rng.permutation(n).astype(np.uint64) + np.uint64(7)
    ctx = q.Context()
    a, b = q.Species(n + 5, dtype), q.Species(n + 9, dtype)
    a.load(x, p, tau, ids)
    grid = torch.zeros(ng ** 3 * 6, dtype=torch.float32, device="cuda")
    print(f"sort: {dtype} n={n}", flush=True)
    ctx.qed_sort_by_cell(q.Fields(q.QED_FIELD_GRID, grid=grid, n=ng, L=L), a, b)
    got = b.to_numpy()
    assert b.n() == n
    back = np.argsort(got["id"])
    order = np.argsort(ids)
    for k, want in (("id", ids), ("x", x), ("p", p), ("tau", tau)):
        assert np.array_equal(got[k][back], want[order])
    ctx.close()


@pytest.mark.parametrize("surrogate", [False, True])
def test_photon_pass_on_a_grid_in_rounds(surrogate):
    """The same where a workgroup takes more than one tile: 4096 tiles of 256 and some
    photons of the next round."""
    test_photon_pass_on_a_grid_staged_equals_global(4096 * 256 + 300, surrogate)


@pytest.mark.parametrize("n", [0, 1, 257, 70_001])
def test_photon_pass_on_a_grid_either_side_of_the_rounds(n):
    """A species whose capacity fills 4096 tiles and one with a tile more: equal ids and
    pairs, positions bit for bit, optical depths to the rounding of a float32 rate
    (two compilations: 64 units in the last place of W dt <= tau's scale of 1)."""
    torch, q = need_gpu()
    ng, L, dt = 32, workloads.BOX_L, 0.01
    rng = np.random.default_rng(n + 2)
    x = rng.uniform(0.0, L, (n, 3))
    k = rng.normal(size=(n, 3))
    k *= (10.0 ** rng.uniform(0.0, 4.0, n) / np.linalg.norm(k, axis=1))[:, None]
    tau, ids = rng.exponential(size=n) * 0.05, np.arange(n, dtype=np.uint64)
    out = []
    for cap in (4096 * 256, 4096 * 256 + 1):
        print(f"photon pass on a grid: n={n} capacity {cap}", flush=True)
        ctx = q.Context(seed=3, kmax=4)
        ctx.qed_build_tables(q.QED_FORMULA_I)
        grid = torch.empty(ng ** 3 * 6, dtype=torch.float32, device="cuda")
        fld = q.Fields(q.QED_FIELD_GRID, grid=grid, n=ng, L=L)
        ctx.qed_fill_standing_wave(grid, ng, L, 1000.0, 0.3)
        ph, el, po = q.Species(cap, "f32"), q.Species(n + 1, "f32"), q.Species(n + 1, "f32")
        ph.load(x, k, tau, ids)
        ctx.qed_set_next_id(n)
        ctx.qed_create_pairs(fld, ph, el, po, dt, 0)
        out.append((ph.to_numpy(), el.to_numpy(), ctx.qed_get_status()[0]))
        ctx.close()
    (pa, ea, sa), (pb, eb, sb) = out
    assert sa == sb and (n < 1000 or sa["pairs"] > 0)
    assert np.array_equal(pa["id"], pb["id"]) and np.array_equal(pa["x"], pb["x"]) and np.array_equal(ea["id"], eb["id"])
    assert np.all(np.abs(pa["tau"] - pb["tau"]) <= ULPS["f32"] * np.maximum(1.0, np.abs(pa["tau"])))
