"""A species as a whole against the same particles in parts, one call after the other:
appends are in particle order and ids follow each other, so ids, counts and order
are equal whatever kernel a size takes and however many tiles a workgroup of it takes;
values agree to the roundings of two compilations of an event (64 units in the last
place)."""
import numpy as np
import pytest

from tests.gpu_helpers import need_gpu

import workloads

pytestmark = pytest.mark.gpu

ULPS = {"f32": 64 * 2.0 ** -24, "f64": 64 * 2.0 ** -53}


def _same(a, b, dtype):
    assert np.array_equal(a["id"], b["id"])
    for k in ("x", "p"):
        scale = np.maximum(np.abs(b[k]), np.abs(b[k]).max(axis=1, keepdims=True))
        assert np.all(np.abs(a[k] - b[k]) <= ULPS[dtype] * scale)
    assert np.all(np.abs(a["tau"] - b["tau"]) <= ULPS[dtype] * np.maximum(1.0, np.abs(b["tau"])))


def _join(parts):
    return {k: np.concatenate([p[k] for p in parts]) for k in parts[0]}


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("method1", [False, True])
@pytest.mark.parametrize("dt", [0.01, 2.0])
def test_emission_whole_equals_parts(dtype, method1, dt):
    """300001 electrons, with dt = 2 nearly all of them emitting: more tiles of the
    list than compute units; parts of up to 2^17, which are emitted without a list."""
    torch, q = need_gpu()
    n, part = 300_001, 1 << 17
    ens = workloads.uniform_b_ensembles(n, seed=5, triples=((2000.0, 206.0),))[0]
    fld = q.Fields(q.QED_FIELD_UNIFORM, B=(0, 0, 2000.0))
    out = []
    for size in (n, part):
        print(f"emission: {dtype} method1={method1} dt={dt} in parts of {size}", flush=True)
        ctx = q.Context(seed=9, kmax=4, flags=q.QED_FLAG_METHOD_I if method1 else 0)
        ctx.qed_build_tables(q.QED_FORMULA_I)
        ctx.qed_set_next_id(n)
        ph, leps = q.Species(4 * n, dtype), []
        for a in range(0, n, size):
            b = min(a + size, n)
            lep = q.Species(b - a, dtype)
            lep.load(ens["x"][a:b], ens["p"][a:b], np.zeros(b - a), ens["id"][a:b])
            ctx.qed_init_optical_depth(lep, 0)
            ctx.qed_gather_push(fld, lep, -1, dt, 0)
            ctx.qed_emit_photons(lep, ph, 0)
            leps.append(lep)
        st, _ = ctx.qed_get_status()
        out.append((_join([s.to_numpy() for s in leps]), ph.to_numpy(), st))
        ctx.close()
    (la, pa, sa), (lb, pb, sb) = out
    assert sa == sb and sa["photons"] == pa["id"].size > 1000 and sa["dropped"] == 0
    _same(la, lb, dtype)
    _same(pa, pb, dtype)


@pytest.mark.parametrize("path", ["f64", "f32", "surrogate"])
@pytest.mark.parametrize("grid", [False, True])
@pytest.mark.parametrize("n,part", [(150_001, 1 << 16), ((1 << 18) - 1, 1 << 17), (300_001, 150_001), (300_001, 1 << 16)])
def test_pairs_whole_equals_parts(path, grid, n, part):
    """A third of the photons convert at once, the others have a step's time.  Float64: one
    photon per thread up to 2^17 and on a grid, two up to 2^18 slots, four above;
    surrogate: more tiles of candidates than the chip holds workgroups."""
    torch, q = need_gpu()
    dtype = "f64" if path == "f64" else "f32"
    ng, L = 16, workloads.BOX_L
    rng = np.random.default_rng(n)
    x = rng.uniform(0.0, L, (n, 3))
    k = rng.normal(size=(n, 3))
    k *= (10.0 ** rng.uniform(2.0, 4.0, n) / np.linalg.norm(k, axis=1))[:, None]
    tau, ids = rng.exponential(size=n) * 0.05, np.arange(n, dtype=np.uint64)
    tau[::3] = 1e-6
    gr = torch.empty(ng ** 3 * 6, dtype=torch.float32, device="cuda")
    out = []
    for size in (n, part):
        print(f"pairs: {path} grid={grid} n={n} in parts of {size}", flush=True)
        ctx = q.Context(seed=2, kmax=4, flags=q.QED_FLAG_SURROGATE if path == "surrogate" else 0)
        ctx.qed_build_tables(q.QED_FORMULA_I)
        if path == "surrogate":             # (weights of any kind: a rate outside the envelope takes the table)
            for net in (0, 1):
                m = q.lib().qed_surrogate_params(net)
                ctx.qed_surrogate_io(net, np.random.default_rng(net).normal(0, 0.05, m).astype(np.float32))
        ctx.qed_fill_standing_wave(gr, ng, L, 2000.0, 0.3)
        fld = (q.Fields(q.QED_FIELD_GRID, grid=gr, n=ng, L=L) if grid
               else q.Fields(q.QED_FIELD_UNIFORM, E=(100.0, -50.0, 30.0), B=(0, 0, 2000.0)))
        ctx.qed_set_next_id(n)
        el, po, phs = q.Species(n, dtype), q.Species(n, dtype), []
        for a in range(0, n, size):
            b = min(a + size, n)
            ph = q.Species(b - a, dtype)
            ph.load(x[a:b], k[a:b], tau[a:b], ids[a:b])
            ctx.qed_create_pairs(fld, ph, el, po, 0.01, 0)
            phs.append(ph)
        st, _ = ctx.qed_get_status()
        out.append(([_join([s.to_numpy() for s in phs]), el.to_numpy(), po.to_numpy()], st))
        ctx.close()
    (a, sa), (b, sb) = out
    assert sa == sb and sa["pairs"] == a[1]["id"].size > n // 20 and sa["dropped"] == 0
    for u, v in zip(a, b):
        _same(u, v, dtype)
