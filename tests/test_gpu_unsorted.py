"""Species in cell order, whose workgroups read the field from a box of nodes in LDS,
against the same particles in random order, whose boxes do not fit, so that they read
it from global memory a stencil row at a time."""
import numpy as np
import pytest

from tests.gpu_helpers import need_gpu

import workloads

pytestmark = pytest.mark.gpu

BOX_NODES = {256: 1024, 512: 2048}


def _fitting(x, ng, L, tile):
    """Share of the tiles of `tile` consecutive positions whose box of stencil nodes
    (rows and planes at odd pitches) has at most BOX_NODES nodes."""
    j = np.floor(x / (L / ng) + 0.5).astype(np.int64) % ng
    fit = []
    for b in range(0, len(j), tile):
        rel = (j[b:b + tile] - j[b] + ng // 2) % ng
        dim = rel.max(0) - rel.min(0) + 3
        row = dim[0] | 1
        fit.append(((row * dim[1]) | 1) * dim[2] <= BOX_NODES[tile])
    return np.mean(fit)


def _context(q, surrogate):
    ctx = q.Context(seed=3, kmax=4, flags=q.QED_FLAG_SURROGATE if surrogate else 0)
    ctx.qed_build_tables(q.QED_FORMULA_I)
    if surrogate:                       # (weights of any kind: a rate outside the envelope takes the table)
        for net in (0, 1):
            m = q.lib().qed_surrogate_params(net)
            ctx.qed_surrogate_io(net, np.random.default_rng(net).normal(0, 0.05, m).astype(np.float32))
    return ctx


@pytest.mark.parametrize("surrogate", [False, True])
@pytest.mark.parametrize("n,capacity,tile", [(600_001, 600_001, 512), (513, 600_001, 512),
                                             (600_001, 5 * 64 ** 3, 256), (257, 5 * 64 ** 3, 256)])
def test_lepton_pass_box_equals_rows(n, capacity, tile, surrogate):
    """Positions within 2 units in the last place of the box length, momenta within 16
    of the larger of |p| and the kick a0 dt, optical depths within the rate's 1e-6."""
    torch, q = need_gpu()
    ng, L, dt, a0 = 64, workloads.BOX_L, 0.01, 500.0
    ens = workloads.standing_wave_electrons(n, seed=8)
    tau = np.random.default_rng(1).exponential(size=n)
    grid = torch.empty(ng ** 3 * 6, dtype=torch.float32, device="cuda")
    fld = q.Fields(q.QED_FIELD_GRID, grid=grid, n=ng, L=L)
    out = []
    for order in ("sorted", "random"):
        print(f"lepton pass: n={n} {order} capacity {capacity} surrogate={surrogate}", flush=True)
        ctx = _context(q, surrogate)
        ctx.qed_fill_standing_wave(grid, ng, L, a0, 0.21)
        lep, ph = q.Species(capacity, "f32"), q.Species(400_000, "f32")
        lep.load(ens["x"], ens["p"], tau, ens["id"])
        if order == "sorted":
            src, lep = lep, q.Species(capacity, "f32")
            ctx.qed_sort_by_cell(fld, src, lep)
        ctx.qed_set_next_id(n)
        if n > 1000:
            fit = _fitting(lep.to_numpy()["x"], ng, L, tile)
            assert fit > 0.5 if order == "sorted" else fit == 0
        ctx.qed_gather_push(fld, lep, -1, dt, 0)
        g = lep.to_numpy()
        ctx.qed_emit_photons(lep, ph, 0)
        st, _ = ctx.qed_get_status()
        if n > 1000:
            tiles = -(-n // tile)
            assert st["box_fallback"] == tiles if order == "random" else st["box_fallback"] < tiles // 2
        k = np.argsort(g["id"])
        out.append(([g[c][k] for c in ("x", "p", "tau")], st["events"] + st["thinned"]))
        ctx.close()
    (a, ea), (b, eb) = out
    assert ea == eb and (n < 1000 or ea > 1000)
    assert np.max(np.abs(a[0] - b[0])) <= 2.0 ** -20
    assert np.max(np.abs(a[1] - b[1]) / np.maximum(np.abs(b[1]), a0 * dt)) <= 2.0 ** -19
    np.testing.assert_allclose(a[2], b[2], rtol=1e-6, atol=1e-6)


@pytest.mark.parametrize("surrogate", [False, True])
@pytest.mark.parametrize("order", ["sorted", "random"])
@pytest.mark.parametrize("n", [0, 1, 257, 4096 * 256 + 300])
def test_photon_pass_in_rounds_of_workgroups(n, order, surrogate):
    """A photon species with 2^24 slots, whose workgroups take more than one tile (4096
    tiles a round), and one with a slot less: equal ids and pairs, positions bit for
    bit, optical depths to the rounding of a float32 rate (two compilations: 64 units
    in the last place of W dt <= tau's scale of 1).  Every third photon dead."""
    torch, q = need_gpu()
    ng, L, dt = 64, workloads.BOX_L, 0.01
    rng = np.random.default_rng(n + 2)
    x = rng.uniform(0.0, L, (n, 3))
    k = rng.normal(size=(n, 3))
    k *= (10.0 ** rng.uniform(0.0, 4.0, n) / np.linalg.norm(k, axis=1))[:, None]
    tau, ids = rng.exponential(size=n) * 0.05, np.arange(n, dtype=np.uint64)
    if order == "sorted":
        cell = np.floor(x / (L / ng) + 0.5).astype(np.int64) % ng
        c = [*cell.T, *(cell // 4).T]
        key = np.lexsort(c)
        x, k, tau = x[key], k[key], tau[key]
    if n > 1000:
        fit = _fitting(x, ng, L, 256)
        assert fit > 0.5 if order == "sorted" else fit == 0
    ids[1::3] = np.uint64(0xFFFFFFFFFFFFFFFF)
    grid = torch.empty(ng ** 3 * 6, dtype=torch.float32, device="cuda")
    fld = q.Fields(q.QED_FIELD_GRID, grid=grid, n=ng, L=L)
    out = []
    for cap in ((1 << 24) - 1, 1 << 24):
        print(f"photon pass: n={n} {order} surrogate={surrogate} capacity {cap}", flush=True)
        ctx = _context(q, surrogate)
        ctx.qed_fill_standing_wave(grid, ng, L, 1000.0, 0.3)
        ph, el, po = q.Species(cap, "f32"), q.Species(n + 1, "f32"), q.Species(n + 1, "f32")
        ph.load(x, k, tau, ids)
        ctx.qed_set_next_id(n)
        ctx.qed_create_pairs(fld, ph, el, po, dt, 0)
        out.append((ph.to_numpy(), el.to_numpy(), ctx.qed_get_status()[0]))
        ctx.close()
    (pa, ea, sa), (pb, eb, sb) = out
    assert sa == sb and (n < 1000 or sa["pairs"] > 0)
    for u, v in ((pa, pb), (ea, eb)):
        assert np.array_equal(u["id"], v["id"])
    assert np.array_equal(pa["x"], pb["x"])
    assert np.all(np.abs(pa["tau"] - pb["tau"]) <= 64 * 2.0 ** -24 * np.maximum(1.0, np.abs(pa["tau"])))
