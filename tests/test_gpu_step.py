"""Parity of the GPU Monte Carlo step against the oracle."""
import math

import numpy as np
import pytest

from oracle import mc, spectra, tables
from oracle.constants import E_S, RATE_UNIT
from tests.gpu_helpers import need_gpu

import workloads

pytestmark = pytest.mark.gpu


def test_init_optical_depth():
    torch, q = need_gpu()
    ctx = q.Context(seed=17)
    sp = q.Species(5000, "f64")
    ids = np.arange(10**9, 10**9 + 4321, dtype=np.uint64)
    sp.load(np.zeros((ids.size, 3)), np.zeros((ids.size, 3)), ids=ids)
    ctx.qed_init_optical_depth(sp, step=3)
    got = sp.to_numpy()["tau"]
    ref = mc.init_tau(ids, seed=17, step=3)
    np.testing.assert_allclose(got, ref, rtol=5e-16, atol=0)   # log differs by <= 1 ulp


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_compact_bitexact(dtype):
    torch, q = need_gpu()
    ctx = q.Context()
    rng = np.random.default_rng(5)
    for n in (0, 1, 1023, 1024, 1025, 70001):
        sp = q.Species(max(n, 1) + 17, dtype)
        x = rng.normal(size=(n, 3))
        p = rng.normal(size=(n, 3))
        tau = rng.uniform(size=n)
        ids = np.arange(n, dtype=np.uint64)
        dead = rng.uniform(size=n) < (0.5 if n % 2 else 0.02)
        ids[dead] = mc.DEAD_ID
        sp.load(x, p, tau, ids)
        ctx.qed_compact(sp)
        st, rc = ctx.qed_get_status()
        got = sp.to_numpy()
        cast = (lambda a: a.astype(np.float32).astype(np.float64)) if dtype == "f32" else (lambda a: a)
        oid, ox, op, otau = mc.compact(ids, cast(x), cast(p), tau)
        assert sp.n() == oid.size
        np.testing.assert_array_equal(got["id"], oid)
        np.testing.assert_array_equal(got["x"], ox)
        np.testing.assert_array_equal(got["p"], op)
        np.testing.assert_array_equal(got["tau"], otau)
        assert st["compacted"] == n - oid.size and st["scan_timeouts"] == 0


def _uniform_run(q, ctx, rad_sampler, n_per, steps, dt=0.01, seed=0, recoil=True):
    """Runs the three uniform-B ensembles on GPU and oracle side by side."""
    ens = workloads.uniform_b_ensembles(n_per, seed=seed)
    results = []
    for k, e in enumerate(ens):
        n = e["id"].size
        lep = q.Species(n, "f64")
        ph = q.Species(n * 4 * steps + 16, "f64")
        tau0 = mc.init_tau(e["id"], seed=seed)
        lep.load(e["x"], e["p"], tau0, e["id"])
        nid = 10**6 * (k + 1)
        ctx.qed_set_next_id(nid)
        fld = q.Fields(q.QED_FIELD_UNIFORM, E=(0, 0, 0), B=(0, 0, e["b0"]))
        E = np.zeros((n, 3))
        B = np.tile([0.0, 0.0, e["b0"]], (n, 1))
        ox, op, otau = e["x"].copy(), e["p"].copy(), tau0.copy()
        oph = []
        for s in range(steps):
            ctx.qed_gather_push(fld, lep, -1, dt, s)
            ctx.qed_emit_photons(lep, ph, s)
            r = mc.lepton_step(ox, op, otau, e["id"], E, B, q=-1.0, dt=dt, step=s, seed=seed,
                               sampler=rad_sampler, next_id=nid, recoil=recoil)
            ox, op, otau, nid = r["x"], r["p"], r["tau"], r["next_id"]
            oph.append(r["photons"])
        st, rc = ctx.qed_get_status()
        assert st["scan_timeouts"] == 0 and st["dropped"] == 0
        results.append((lep.to_numpy(), ph.to_numpy(), dict(x=ox, p=op, tau=otau), oph, nid,
                        ctx.qed_get_next_id()))
    return results


def test_uniform_field_f64_parity(rad_table_I):
    """Three Fig. 1 ensembles, float64 state: positions, momenta, optical depths,
    photon lists (order, ids, energies, optical depths) against the oracle."""
    torch, q = need_gpu()
    ctx = q.Context(seed=0, kmax=4)
    ctx.qed_build_tables(q.QED_FORMULA_I)
    rad = mc.RadSampler(rad_table_I, "f64")
    for g, gph, o, oph, nid, gnid in _uniform_run(q, ctx, rad, 3000, 12):
        np.testing.assert_allclose(g["p"], o["p"], rtol=1e-11, atol=1e-9)
        np.testing.assert_allclose(g["x"], o["x"], rtol=1e-11, atol=1e-9)
        np.testing.assert_allclose(g["tau"], o["tau"], rtol=1e-9, atol=1e-9)
        ph_ref = {k: np.concatenate([p[k] for p in oph]) for k in ("x", "k", "tau", "id")}
        assert gph["id"].size == ph_ref["id"].size and nid == gnid
        np.testing.assert_array_equal(gph["id"], ph_ref["id"])
        np.testing.assert_allclose(gph["p"], ph_ref["k"], rtol=1e-10, atol=1e-9)
        np.testing.assert_allclose(gph["tau"], ph_ref["tau"], rtol=1e-12)
        np.testing.assert_allclose(gph["x"], ph_ref["x"], rtol=1e-11, atol=1e-9)


def test_f32_chi_where_fields_cancel(rad_table_I):
    """Float32 path, chi (Eq. 2) where E + v x B nearly cancels: a uniform crossed
    field E = E0 y, B = E0 z (a plane wave moving along +x) and electrons moving
    within 1e-2 rad of +x (chi ~ gamma (1 - beta) E0 / E_S, down to ~2e-6) or of -x
    (chi up to ~20).  The rate each electron applied to its optical depth,
    W = (tau0 - tau1) / dt, is compared with the oracle's rate (the same table) at
    the oracle's chi of the GPU's pushed float32 momentum; a float32 evaluation
    of Eq. 2 would be off by ~1e-7 gamma^2 in the co-moving half.  The oracle's
    float64 chi is itself checked against an 80-bit evaluation of Eq. 2."""
    torch, q = need_gpu()
    rng = np.random.default_rng(5)
    n, E0, dt, tau0 = 20000, 2000.0, 1e-3, 50.0
    gam = 10.0 ** rng.uniform(1.0, 3.0, n)
    th = rng.uniform(0.0, 1e-2, n) * np.where(np.arange(n) % 2 == 0, 1.0, 0.0)
    th[np.arange(n) % 4 == 1] = 0.0
    ph = rng.uniform(0.0, 2.0 * math.pi, n)
    sgn = np.where(np.arange(n) % 4 == 3, -1.0, 1.0)     # a quarter counter-propagating
    pa = np.sqrt(gam ** 2 - 1.0)
    p = np.stack([sgn * pa * np.cos(th), pa * np.sin(th) * np.cos(ph), pa * np.sin(th) * np.sin(ph)], -1)
    p = p.astype(np.float32).astype(np.float64)
    ctx = q.Context(seed=2, kmax=4)
    ctx.qed_build_tables(q.QED_FORMULA_I)
    lep = q.Species(n, "f32")
    ids = np.arange(n, dtype=np.uint64)
    lep.load(np.zeros((n, 3)), p, np.full(n, tau0), ids)
    ctx.qed_set_next_id(n)
    fld = q.Fields(q.QED_FIELD_UNIFORM, E=(0.0, E0, 0.0), B=(0.0, 0.0, E0))
    ctx.qed_gather_push(fld, lep, -1, dt, 0)
    st, _ = ctx.qed_get_status()
    g = lep.to_numpy()
    assert st["events"] == 0 and st["nan_chi"] == 0
    w_gpu = (tau0 - g["tau"]) / dt
    p1 = g["p"]
    E = np.tile([0.0, E0, 0.0], (n, 1))
    B = np.tile([0.0, 0.0, E0], (n, 1))
    chi = spectra.chi_lepton(p1, E, B)
    # 80-bit reference of Eq. 2 on the same inputs
    pl = p1.astype(np.longdouble)
    gl = np.sqrt(1 + np.sum(pl * pl, -1))
    vl = pl / gl[:, None]
    fl = E.astype(np.longdouble) + np.cross(vl, B.astype(np.longdouble))
    chil = gl / E_S * np.sqrt(np.sum(fl * fl, -1) - np.sum(vl * E, -1) ** 2)
    assert np.max(np.abs(chi / chil.astype(np.float64) - 1.0)) < 1e-9
    assert chi.min() < 1e-5 and chi.max() > 5.0
    w_ref = tables.rate_rad(rad_table_I, chi, np.sqrt(1.0 + np.sum(p1 * p1, -1)))
    rel = np.abs(w_gpu / w_ref - 1.0)
    print(f"chi {chi.min():.2e} .. {chi.max():.2e}; rate rel. error max {rel.max():.2e} (co-moving "
          f"{rel[sgn > 0].max():.2e})")
    assert rel.max() < 2e-5


def test_thinned_pass_envelope_where_fields_cancel(rad_table_I):
    """Surrogate path (Poisson thinning): the lepton pass runs the optical depth
    down at the envelope rate alpha E_S h_env(chi_b) / gamma at a float32 upper
    bound chi_b of chi, and thinning is exact only if that envelope is never below
    the rate.  Same crossed-field geometry as above (chi from ~2e-6 co-moving to
    ~20 counter-propagating, no events: tau0 = 50): the applied rate
    (tau0 - tau1) / dt is at or above the oracle's rate at the oracle's chi of the
    pushed momentum for every electron, at or above the envelope at that chi
    (within the float32 evaluation of the envelope, 2e-5), and within 1e-4 of it
    for the counter-propagating electrons, where nothing cancels."""
    torch, q = need_gpu()
    rng = np.random.default_rng(6)
    n, E0, dt, tau0 = 20000, 2000.0, 1e-3, 50.0
    gam = 10.0 ** rng.uniform(1.0, 3.0, n)
    th = rng.uniform(0.0, 1e-2, n) * np.where(np.arange(n) % 2 == 0, 1.0, 0.0)
    th[np.arange(n) % 4 == 1] = 0.0
    ph = rng.uniform(0.0, 2.0 * math.pi, n)
    sgn = np.where(np.arange(n) % 4 == 3, -1.0, 1.0)
    pa = np.sqrt(gam ** 2 - 1.0)
    p = np.stack([sgn * pa * np.cos(th), pa * np.sin(th) * np.cos(ph), pa * np.sin(th) * np.sin(ph)], -1)
    p = p.astype(np.float32).astype(np.float64)
    ctx = q.Context(seed=2, kmax=4, flags=q.QED_FLAG_SURROGATE)
    ctx.qed_build_tables(q.QED_FORMULA_I)
    for net in (0, 1):                              # any weights: the pass uses the envelope only
        rng0 = np.random.default_rng(net)
        ctx.qed_surrogate_io(net, rng0.normal(0, 0.3, q.lib().qed_surrogate_params(net)).astype(np.float32))
    lep = q.Species(n, "f32")
    lep.load(np.zeros((n, 3)), p, np.full(n, tau0), np.arange(n, dtype=np.uint64))
    ctx.qed_set_next_id(n)
    fld = q.Fields(q.QED_FIELD_UNIFORM, E=(0.0, E0, 0.0), B=(0.0, 0.0, E0))
    print(f"thinned lepton pass, crossed field E0 = {E0}, {n} electrons", flush=True)
    ctx.qed_gather_push(fld, lep, -1, dt, 0)
    st, _ = ctx.qed_get_status()
    g = lep.to_numpy()
    assert st["nan_chi"] == 0
    assert np.all(g["tau"] > 0.0)                 # no candidate within the step
    w_gpu = (tau0 - g["tau"]) / dt
    p1 = g["p"]
    gamma1 = np.sqrt(1.0 + np.sum(p1 * p1, -1))
    chi = spectra.chi_lepton(p1, np.tile([0.0, E0, 0.0], (n, 1)), np.tile([0.0, 0.0, E0], (n, 1)))
    assert chi.min() < 1e-5 and chi.max() > 5.0
    w_rate = tables.rate_rad(rad_table_I, chi, gamma1)
    c1 = 5.0 / (2.0 * math.sqrt(3.0))
    w_env = RATE_UNIT * 1.002 * c1 * chi * (1.0 + chi) ** (-1.0 / 3.0) / gamma1
    infl = w_gpu / w_env
    print(f"  applied / envelope at chi: min {infl.min():.6f}, counter-propagating max "
          f"{infl[sgn < 0].max():.6f}, co-moving max {infl[sgn > 0].max():.3e}")
    assert np.all(w_gpu >= w_rate)
    assert infl.min() > 1.0 - 2e-5
    assert infl[sgn < 0].max() < 1.0 + 1e-4


@pytest.mark.parametrize("cap", [2000, 40_000], ids=["one_per_thread", "two_per_thread"])
def test_thinned_pass_on_a_grid(rad_table_I, cap):
    """Surrogate path on a grid (standing wave a0 = 500, 8^3 grid, 1537 electrons,
    tau0 = 50: no candidate within the step), with the species sized for the
    one-particle and for the two-particle lepton kernel: the push against the
    oracle step on the same float32 inputs (the bars of the one-step parity
    test), and the applied rate (tau0 - tau1) / dt at or above the oracle's rate
    at the oracle's chi of the pushed momentum, at or above the envelope at that
    chi (2e-5: the float32 gather and envelope), and at most the envelope at the
    bound the float32 evaluation of chi guarantees for the kernel's own fields
    (chi^2 E_S^2 + 32u (|A|^2 + S^2), u = 2^-24, A and S the sums of magnitudes
    of the terms of a = gamma E + p x B and s = p.E), those fields being within
    28u a0 per component of the oracle's (27 weighted nodes of magnitude <= a0,
    weights summing to 1), which moves |a| by up to sqrt(3) (gamma + |p|) 28u a0
    and |s| by up to sqrt(3) |p| 28u a0; 1e-5 to spare for the float32 envelope."""
    torch, q = need_gpu()
    ng, a0, L, dt, t, n, tau0 = 8, 500.0, workloads.BOX_L, 0.01, 0.37, 1537, 50.0
    ens, x, p = _c2_setup(q, n)
    ctx = q.Context(seed=1, kmax=4, flags=q.QED_FLAG_SURROGATE)
    ctx.qed_build_tables(q.QED_FORMULA_I)
    for net in (0, 1):                              # any weights: the pass uses the envelope only
        rng0 = np.random.default_rng(net)
        ctx.qed_surrogate_io(net, rng0.normal(0, 0.3, q.lib().qed_surrogate_params(net)).astype(np.float32))
    grid = torch.empty(ng ** 3 * 6, dtype=torch.float32, device="cuda")
    ctx.qed_fill_standing_wave(grid, ng, L, a0, t)
    fld = q.Fields(q.QED_FIELD_GRID, grid=grid, n=ng, L=L)
    lep = q.Species(cap, "f32")
    tau = np.full(n, tau0)
    lep.load(x, p, tau, ens["id"])
    ctx.qed_set_next_id(n)
    print(f"thinned pass on a grid, capacity {cap}", flush=True)
    ctx.qed_gather_push(fld, lep, -1, dt, 5)
    st, _ = ctx.qed_get_status()
    g = lep.to_numpy()
    assert st["nan_chi"] == 0 and np.all(g["tau"] > 0.0)
    Eg, Bg = mc.standing_wave_grid(ng, L, a0, t)
    E, B = mc.gather_tsc(Eg, Bg, L, x)
    rad = mc.RadSampler(rad_table_I, "q16")
    r = mc.lepton_step(x, p, tau, ens["id"], E, B, q=-1.0, dt=dt, step=5, seed=1, sampler=rad, next_id=n, L=L)
    assert r["n_events"] == 0
    np.testing.assert_allclose(g["p"], r["p"], rtol=2e-5, atol=2e-5 * np.abs(r["p"]).max())
    dx = np.abs(g["x"] - r["x"])
    assert np.minimum(dx, L - dx).max() < 1e-5
    p1 = g["p"]
    gamma1 = np.sqrt(1.0 + np.sum(p1 * p1, -1))
    chi = spectra.chi_lepton(p1, E, B)
    w_rate = tables.rate_rad(rad_table_I, chi, gamma1)
    c1 = 5.0 / (2.0 * math.sqrt(3.0))

    def env(c):
        return RATE_UNIT * 1.002 * c1 * c * (1.0 + c) ** (-1.0 / 3.0) / gamma1

    px, py, pz = p1[:, 0], p1[:, 1], p1[:, 2]
    ge = np.abs(gamma1[:, None] * E)
    A2 = ((ge[:, 0] + np.abs(py * B[:, 2]) + np.abs(pz * B[:, 1])) ** 2
          + (ge[:, 1] + np.abs(pz * B[:, 0]) + np.abs(px * B[:, 2])) ** 2
          + (ge[:, 2] + np.abs(px * B[:, 1]) + np.abs(py * B[:, 0])) ** 2)
    S2 = np.sum(np.abs(p1 * E), -1) ** 2
    u = 2.0 ** -24
    pa = np.linalg.norm(p1, axis=1)
    a_mag = np.linalg.norm(gamma1[:, None] * E + np.cross(p1, B), axis=1)
    s_mag = np.abs(np.sum(p1 * E, -1))
    da = math.sqrt(3.0) * (gamma1 + pa) * 28.0 * u * a0
    ds = math.sqrt(3.0) * pa * 28.0 * u * a0
    gather = 2.0 * a_mag * da + da ** 2 + 2.0 * s_mag * ds + ds ** 2
    chi_hi = np.sqrt(chi ** 2 + (32.0 * u * (A2 + S2) + gather) / E_S ** 2) * (1.0 + 2.0 ** -20)
    w_gpu = (tau0 - g["tau"]) / dt
    lo, hi = w_gpu / env(chi), w_gpu / env(chi_hi)
    print(f"  chi {chi.min():.2e} .. {chi.max():.2e}; applied / envelope at chi {lo.min():.6f} .. {lo.max():.6f}, "
          f"at the bound max {hi.max():.6f}")
    assert np.all(w_gpu >= w_rate)
    assert lo.min() > 1.0 - 2e-5 and hi.max() < 1.0 + 1e-5


def _chi_ref80(p, E, B, photon):
    """Eq. (2) (or Eq. (3) with |v| = 1) evaluated literally in 80-bit floats."""
    pl, El, Bl = (a.astype(np.longdouble) for a in (p, E, B))
    pa = np.sqrt(np.sum(pl * pl, -1))
    g = pa if photon else np.sqrt(1 + pa * pa)
    v = pl / (pa if photon else g)[:, None]
    f = El + np.cross(v, Bl)
    return (g / E_S * np.sqrt(np.maximum(np.sum(f * f, -1) - np.sum(v * El, -1) ** 2, 0))).astype(np.float64)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_chi_vs_oracle_1e6(dtype):
    """qed_eval_chi (the step's chi code) against the oracle's Eq. (2) / Eq. (3)
    on the same inputs, relative error <= 1e-6, in the geometries where
    E + v x B cancels: a crossed field E0 y, E0 z (a plane wave along +x) with
    leptons within 1e-2 rad of +x (chi ~ gamma (1 - beta) E0 / E_S, down to ~1e-7)
    and of -x, gamma 10 .. 1e4; random momenta in random per-particle fields; photons
    isotropic and 1e-3 .. 1e-2 rad from +x in the crossed field.  The oracle's literal
    float64 form is itself checked against an 80-bit evaluation (its error grows as
    3e-16 gamma^2, R15, below 3e-8 here)."""
    torch, q = need_gpu()
    rng = np.random.default_rng(8)
    cast = (lambda a: a.astype(np.float32).astype(np.float64)) if dtype == "f32" else (lambda a: a)
    ctx = q.Context(seed=2)
    n, E0 = 40000, 2000.0
    gam = 10.0 ** rng.uniform(1.0, 4.0, n)
    th = rng.uniform(0.0, 1e-2, n)
    ph = rng.uniform(0.0, 2 * math.pi, n)
    sgn = np.where(np.arange(n) % 4 == 3, -1.0, 1.0)
    pa = np.sqrt(gam ** 2 - 1.0)
    p_x = cast(np.stack([sgn * pa * np.cos(th), pa * np.sin(th) * np.cos(ph), pa * np.sin(th) * np.sin(ph)], -1))
    p_r = cast(rng.normal(size=(n, 3)) * (10.0 ** rng.uniform(0, 4, n))[:, None])
    f32 = lambda a: a.astype(np.float32).astype(np.float64)   # field arrays are float32 in the ABI
    E_r = f32(rng.uniform(-2000, 2000, (n, 3)))
    B_r = f32(rng.uniform(-2000, 2000, (n, 3)))
    k_iso = rng.normal(size=(n, 3))
    k_iso = cast(k_iso / np.linalg.norm(k_iso, axis=1)[:, None] * (10.0 ** rng.uniform(0, 5, n))[:, None])
    # photons: chi_ph ~ gamma (1 - cos th) E0 / E_S; the literal form loses ~1/th^2 of
    # its digits to cancellation, so th >= 1e-3 keeps the oracle itself within 1e-7
    th2 = rng.uniform(1e-3, 1e-2, n)
    k_x = cast(np.stack([np.cos(th2), np.sin(th2) * np.cos(ph), np.sin(th2) * np.sin(ph)], -1) * gam[:, None])
    Ec, Bc = np.tile([0.0, E0, 0.0], (n, 1)), np.tile([0.0, 0.0, E0], (n, 1))
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()
    crossed = q.Fields(q.QED_FIELD_UNIFORM, E=(0.0, E0, 0.0), B=(0.0, 0.0, E0))
    perpart = q.Fields(q.QED_FIELD_PER_PARTICLE, E=[dev(E_r[:, c]) for c in range(3)],
                       B=[dev(B_r[:, c]) for c in range(3)])
    out = torch.empty(n, dtype=torch.float64, device="cuda")
    cases = (("lepton, crossed field", p_x, crossed, Ec, Bc, False),
             ("lepton, random fields", p_r, perpart, E_r, B_r, False),
             ("photon, random fields", k_iso, perpart, E_r, B_r, True),
             ("photon, near the wave vector", k_x, crossed, Ec, Bc, True))
    for name, p, fld, E, B, photon in cases:
        sp = q.Species(n, dtype)
        sp.load(np.zeros((n, 3)), p)
        print(f"chi {dtype}: {name}", flush=True)
        ctx.qed_eval_chi(fld, sp, q.QED_CHI_PHOTON if photon else q.QED_CHI_LEPTON, out)
        torch.cuda.synchronize()
        got = out.cpu().numpy()
        ref = spectra.chi_photon(p, E, B) if photon else spectra.chi_lepton(p, E, B)
        ref80 = _chi_ref80(p, E, B, photon)
        pos = ref80 > 0
        assert np.max(np.abs(ref[pos] / ref80[pos] - 1)) < 1e-7
        rel = np.abs(got[pos] / ref[pos] - 1)
        print(f"  chi {ref[pos].min():.2e} .. {ref.max():.2e}: max rel err {rel.max():.2e}")
        assert rel.max() <= 1e-6
        assert np.all(got[~pos] <= 1e-9 * ref.max())


def test_fill_standing_wave_vs_oracle():
    """qed_fill_standing_wave on even (float4 stores) and odd (float2 stores) grids,
    and from a grid pointer that is only 8-byte aligned: every node against the
    oracle's node values (float32 rounding of float64 values)."""
    torch, q = need_gpu()
    ctx = q.Context(seed=0)
    L, a0 = workloads.BOX_L, 500.0
    for n, t, off in ((128, 0.37, 0), (5, 1.1, 0), (6, 2.3, 2)):
        buf = torch.full((n ** 3 * 6 + 4,), float("nan"), dtype=torch.float32, device="cuda")
        grid = buf[off:off + n ** 3 * 6]            # off = 2 floats: 8-byte but not 16-byte aligned
        ctx.qed_fill_standing_wave(grid, n, L, a0, t)
        g = grid.cpu().numpy().reshape(n, n, n, 6)   # [iz, iy, ix, component]
        Eg, Bg = mc.standing_wave_grid(n, L, a0, t)  # [c, ix, iy, iz]
        ref = np.concatenate([Eg, Bg], 0).transpose(3, 2, 1, 0)
        np.testing.assert_allclose(g, ref, rtol=2e-7, atol=2e-7 * a0)
        assert np.isnan(buf[:off].cpu().numpy()).all() and np.isnan(buf[off + n ** 3 * 6:].cpu().numpy()).all()
    ctx.close()


def test_uniform_b_full_size_subsample(rad_table_I):
    """Configuration 1 at full size: the three Fig. 1 ensembles of 1e5 electrons
    each, float64, formula I, 100 steps of dt = 0.01, seed 0, optical depths drawn
    on the GPU.  The first 2000 electrons of each ensemble end in the same state
    as the oracle run on those electrons alone (particles are independent and
    their streams depend on their ids only); photons per electron agree within
    4 sigma; photon energies pass a two-sample KS test at the 0.1 % level."""
    torch, q = need_gpu()
    n_per, steps, sub, dt = 100000, 100, 2000, 0.01
    ctx = q.Context(seed=0, kmax=4)
    ctx.qed_build_tables(q.QED_FORMULA_I)
    rad = mc.RadSampler(rad_table_I, "f64")
    for k, e in enumerate(workloads.uniform_b_ensembles(n_per, seed=0)):
        n = e["id"].size
        lep = q.Species(n, "f64")
        ph = q.Species(n * 16, "f64")
        lep.load(e["x"], e["p"], None, e["id"])
        ctx.qed_init_optical_depth(lep, 0)
        ctx.qed_set_next_id(10**7 * (k + 1))
        fld = q.Fields(q.QED_FIELD_UNIFORM, E=(0, 0, 0), B=(0, 0, e["b0"]))
        for s in range(steps):
            ctx.qed_gather_push(fld, lep, -1, dt, s)
            ctx.qed_emit_photons(lep, ph, s)
        st, rc = ctx.qed_get_status()
        # kmax = 4 events per step is reached a handful of times (Poisson tail at
        # W dt ~ 0.15 over 1e7 particle-steps); the oracle caps the same way
        assert st["scan_timeouts"] == 0 and st["dropped"] == 0
        g = lep.to_numpy()
        gph = np.linalg.norm(ph.to_numpy()["p"], axis=1)
        ids = e["id"][:sub]
        ox, op, otau = e["x"][:sub].copy(), e["p"][:sub].copy(), mc.init_tau(ids, seed=0)
        E = np.zeros((sub, 3))
        B = np.tile([0.0, 0.0, e["b0"]], (sub, 1))
        oph = []
        for s in range(steps):
            r = mc.lepton_step(ox, op, otau, ids, E, B, q=-1.0, dt=dt, step=s, seed=0, sampler=rad,
                               next_id=0)
            ox, op, otau = r["x"], r["p"], r["tau"]
            oph.append(np.linalg.norm(r["photons"]["k"], axis=1))
        oph = np.concatenate(oph)
        np.testing.assert_array_equal(g["id"][:sub], ids)
        np.testing.assert_allclose(g["p"][:sub], op, rtol=1e-9, atol=1e-9)
        np.testing.assert_allclose(g["x"][:sub], ox, rtol=1e-9, atol=1e-9)
        np.testing.assert_allclose(g["tau"][:sub], otau, rtol=1e-8, atol=1e-8)
        a, b = gph.size / n, oph.size / sub
        print(f"ensemble {k}: photons per electron GPU {a:.4f} (n={gph.size}) oracle subsample {b:.4f} "
              f"(n={oph.size})")
        assert abs(a - b) < 4 * math.sqrt(oph.size) / sub
        ga, gb = np.sort(gph), np.sort(oph)
        allv = np.concatenate([ga, gb])
        ks = np.max(np.abs(np.searchsorted(ga, allv, side="right") / ga.size
                           - np.searchsorted(gb, allv, side="right") / gb.size))
        assert ks < 1.95 * math.sqrt((ga.size + gb.size) / (ga.size * gb.size))


def test_sample_entry_point(rad_table_I, pair_table):
    torch, q = need_gpu()
    ctx = q.Context(seed=4)
    ctx.qed_build_tables(q.QED_FORMULA_I)
    inp = workloads.sampler_inputs(200000, seed=3)
    chi = np.concatenate([inp["chi"], [1e-6, 5e-4, 1e-3, 99.9, 100.0, 300.0]])
    gam = np.concatenate([inp["gamma"], [1e3] * 6])
    ids = np.arange(chi.size, dtype=np.uint64)
    dev = lambda a, dt: torch.from_numpy(a).to("cuda", dt)
    tchi, tg = dev(chi, torch.float64), dev(gam, torch.float64)
    tid = dev(ids.view(np.int64), torch.int64)
    from oracle import philox
    r = philox.stream(ids, 4, 7, philox.LEPTON_EVENT, 0)
    u = philox.uniform(r)
    for prec, storage, rtol_w, tol_s in ((q.QED_F64, "f64", 1e-6, 1e-10), (q.QED_F32, "q16", 2e-5, 3e-3)):
        lnw = torch.empty(chi.size, dtype=torch.float32, device="cuda")
        xi = torch.empty_like(lnw)
        lnwp = torch.empty_like(lnw)
        ctx.qed_sample(tchi, tg, tid, prec, 7, lnw, xi, lnwp)
        torch.cuda.synchronize()
        rs = mc.RadSampler(rad_table_I, storage)
        ps = mc.PairSampler(pair_table, storage)
        w_ref = rs.rate(chi, gam)
        np.testing.assert_allclose(np.exp(lnw.cpu().numpy().astype(np.float64)), w_ref, rtol=rtol_w)
        wp = ps.rate(chi, gam)
        ok = wp > 1e-30
        np.testing.assert_allclose(np.exp(lnwp.cpu().numpy().astype(np.float64))[ok], wp[ok], rtol=rtol_w * 10)
        xr, _ = rs.sample(chi, u[:, 0], u[:, 2])
        xg = xi.cpu().numpy().astype(np.float64)
        # tol_s is the logit tolerance of the table copy; the output is float32
        lim = tol_s * xr * (1 - xr) + 1.2e-7 * xr
        assert np.all(np.abs(xg - xr) <= lim), np.max(np.abs(xg - xr) / lim)


def _c2_setup(q, n, seed=1, a0=500.0, ngrid=128):
    ens = workloads.standing_wave_electrons(n, seed=seed)
    x32 = ens["x"].astype(np.float32).astype(np.float64)
    p32 = ens["p"].astype(np.float32).astype(np.float64)
    return ens, x32, p32


@pytest.mark.parametrize("ngrid,cap", [(128, None), (32, 2_200_000)], ids=["one_per_thread", "two_per_thread"])
def test_grid_step_f32_one_step_parity(rad_table_I, ngrid, cap):
    """Standing wave a0 = 500, float32 state: one step per particle against the
    oracle (float64 arithmetic on the same float32 inputs), on a 128^3 grid with a
    species of 1e5 (one particle per thread) and on a 32^3 grid with a species
    sized for 2.2e6 (two per thread: at least 64 per cell) holding the same 1e5."""
    torch, q = need_gpu()
    n, a0, L, dt = 100000, 500.0, workloads.BOX_L, 0.01
    ctx = q.Context(seed=1, kmax=4)
    ctx.qed_build_tables(q.QED_FORMULA_I)
    ens, x, p = _c2_setup(q, n)
    tau = mc.init_tau(ens["id"], seed=1)
    # give half of the particles a small optical depth so that many emit
    tau[::2] *= 1e-3
    grid = torch.empty(ngrid ** 3 * 6, dtype=torch.float32, device="cuda")
    print(f"grid step parity: {ngrid}^3, capacity {cap or n}", flush=True)
    lep = q.Species(cap or n, "f32")
    ph = q.Species(4 * n, "f32")
    lep.load(x, p, tau, ens["id"])
    ctx.qed_set_next_id(n)
    t = 0.37
    ctx.qed_fill_standing_wave(grid, ngrid, L, a0, t)
    fld = q.Fields(q.QED_FIELD_GRID, grid=grid, n=ngrid, L=L)
    ctx.qed_gather_push(fld, lep, -1, dt, 5)
    ctx.qed_emit_photons(lep, ph, 5)
    st, rc = ctx.qed_get_status()
    g = lep.to_numpy()
    gph = ph.to_numpy()
    Eg, Bg = mc.standing_wave_grid(ngrid, L, a0, t)
    E, B = mc.gather_tsc(Eg, Bg, L, x)
    rad = mc.RadSampler(rad_table_I, "q16")
    r = mc.lepton_step(x, p, tau, ens["id"], E, B, q=-1.0, dt=dt, step=5, seed=1, sampler=rad,
                       next_id=n, L=L)
    # decisions: the first-event decision tau <= W dt of a particle can flip only
    # if its margin is below the float32 rate error (1e-5 of W dt: the hardware
    # log/exp of the table lookup, ~1e-6, and the float32 push); the event
    # counts must agree exactly unless such particles exist
    W = r["W"]
    ambiguous = int(np.count_nonzero(np.abs(tau - W * dt) <= 1e-5 * W * dt))
    print(f"events GPU {st['events']} oracle {r['n_events']}, ambiguous decisions {ambiguous}")
    assert abs(st["events"] - r["n_events"]) <= 4 * ambiguous and st["scan_timeouts"] == 0
    np.testing.assert_allclose(g["p"], r["p"], rtol=2e-5, atol=2e-5 * np.abs(r["p"]).max())
    dx = np.abs(g["x"] - r["x"])
    dx = np.minimum(dx, L - dx)
    assert dx.max() < 1e-5
    assert gph["id"].size == r["photons"]["id"].size
    np.testing.assert_array_equal(gph["id"], r["photons"]["id"])
    # gamma_ph: both sides decode the same 16-bit quantiles; float32 interpolation
    # and decode stay far below the 16-bit step (<= 3e-4 relative in xi)
    gerr = np.abs(np.linalg.norm(gph["p"], axis=1) / r["photons"]["gamma"] - 1)
    print(f"gamma_ph max rel err {gerr.max():.2e}")
    assert gerr.max() <= 3e-4
    np.testing.assert_allclose(gph["tau"], r["photons"]["tau"], rtol=1e-12)
    np.testing.assert_allclose(g["tau"], r["tau"], rtol=2e-4, atol=2e-4 * (W * dt).max())


def test_two_per_thread_small_and_ragged_counts(rad_table_I):
    """The two-particle lepton pass (a species sized for at least 64 particles
    per cell: capacity 40000 on an 8^3 grid) at counts that leave tiles partly
    empty: none, one, the first half of a 512-particle tile and one more, a whole
    tile and one more, three tiles and one more.  Each count against the oracle
    step on the same float32 inputs (events, momenta, positions, photon ids and
    energies), to the bars of the one-step parity test."""
    torch, q = need_gpu()
    ng, a0, L, dt, t = 8, 500.0, workloads.BOX_L, 0.01, 0.37
    ens, x_all, p_all = _c2_setup(q, 1537)
    tau_all = mc.init_tau(ens["id"], seed=1)
    tau_all[::2] *= 1e-3
    grid = torch.empty(ng ** 3 * 6, dtype=torch.float32, device="cuda")
    Eg, Bg = mc.standing_wave_grid(ng, L, a0, t)
    rad = mc.RadSampler(rad_table_I, "q16")
    for n in (0, 1, 256, 257, 512, 513, 1537):
        print(f"two per thread, {n} electrons", flush=True)
        ctx = q.Context(seed=1, kmax=4)
        ctx.qed_build_tables(q.QED_FORMULA_I)
        ctx.qed_fill_standing_wave(grid, ng, L, a0, t)
        fld = q.Fields(q.QED_FIELD_GRID, grid=grid, n=ng, L=L)
        lep = q.Species(40_000, "f32")
        ph = q.Species(8192, "f32")
        x, p, tau, ids = x_all[:n], p_all[:n], tau_all[:n], ens["id"][:n]
        if n:
            lep.load(x, p, tau, ids)
        ctx.qed_set_next_id(n)
        ctx.qed_gather_push(fld, lep, -1, dt, 5)
        ctx.qed_emit_photons(lep, ph, 5)
        st, rc = ctx.qed_get_status()
        assert st["scan_timeouts"] == 0 and st["dropped"] == 0
        if n == 0:
            assert lep.n() == 0 and ph.n() == 0 and st["events"] == 0
            ctx.close()
            continue
        g, gph = lep.to_numpy(), ph.to_numpy()
        E, B = mc.gather_tsc(Eg, Bg, L, x)
        r = mc.lepton_step(x, p, tau, ids, E, B, q=-1.0, dt=dt, step=5, seed=1, sampler=rad, next_id=n, L=L)
        W = r["W"]
        ambiguous = int(np.count_nonzero(np.abs(tau - W * dt) <= 1e-5 * W * dt))
        assert abs(st["events"] - r["n_events"]) <= 4 * ambiguous
        np.testing.assert_array_equal(g["id"], ids)
        np.testing.assert_allclose(g["p"], r["p"], rtol=2e-5, atol=2e-5 * np.abs(r["p"]).max())
        dx = np.abs(g["x"] - r["x"])
        assert np.minimum(dx, L - dx).max() < 1e-5
        np.testing.assert_array_equal(gph["id"], r["photons"]["id"])
        if gph["id"].size:
            gerr = np.abs(np.linalg.norm(gph["p"], axis=1) / r["photons"]["gamma"] - 1)
            assert gerr.max() <= 3e-4
        np.testing.assert_allclose(g["tau"], r["tau"], rtol=2e-4, atol=2e-4 * (W * dt).max())
        ctx.close()


def test_emitted_spectrum_ks_1e7(rad_table_I):
    """Fixed chi ~ 1 (Fig. 1 b), no recoil, float32 path: 1e7 emitted photons.
    xi against the exact truncated CDF (one-sample KS) and against the oracle's
    table sampler (two-sample KS), both <= 2e-3."""
    torch, q = need_gpu()
    n, b0, g = 1_000_000, 2000.0, 206.0
    ctx = q.Context(seed=21, kmax=4, flags=q.QED_FLAG_NO_RECOIL)
    ctx.qed_build_tables(q.QED_FORMULA_I)
    ens = workloads.uniform_b_ensembles(n, seed=21, triples=((b0, g),))[0]
    lep = q.Species(n, "f32")
    ph = q.Species(12_000_000, "f32")
    lep.load(ens["x"], ens["p"], ids=ens["id"])
    ctx.qed_init_optical_depth(lep, 0)
    ctx.qed_set_next_id(n)
    fld = q.Fields(q.QED_FIELD_UNIFORM, B=(0, 0, b0))
    s = 0
    while ph.n() < 10_000_000:
        ctx.qed_gather_push(fld, lep, -1, 0.05, s)
        ctx.qed_emit_photons(lep, ph, s)
        s += 1
    st, rc = ctx.qed_get_status()
    assert st["dropped"] == 0 and st["scan_timeouts"] == 0
    nph = ph.n()
    gam = torch.sqrt(ph.px[:nph].double() ** 2 + ph.py[:nph].double() ** 2 + ph.pz[:nph].double() ** 2)
    xi = np.sort((gam / g).cpu().numpy())
    chi = g * math.sqrt(1 - 1 / g ** 2) * b0 / E_S
    row = tables.fine_row("I", chi, tables.RAD_M)
    P = row.F / row.total
    xc = 2.0 / g
    Pc = float(np.interp(math.log(xc) - math.log1p(-xc), row.s, P))
    Pe = (np.interp(np.log(xi) - np.log1p(-np.minimum(xi, 1 - 1e-7)), row.s, P) - Pc) / (1 - Pc)
    m = xi.size
    ks1 = max(np.max(np.arange(1, m + 1) / m - Pe), np.max(Pe - np.arange(m) / m))
    # oracle sampler (same 16-bit table copy), same number of accepted samples
    rng = np.random.default_rng(99)
    want = m
    got = []
    rs = mc.RadSampler(rad_table_I, "q16")
    while sum(a.size for a in got) < want:
        u = (np.floor(rng.uniform(size=4_000_000) * 2 ** 23) + 0.5) * 2.0 ** -23
        ur = (np.floor(rng.uniform(size=4_000_000) * 2 ** 23) + 0.5) * 2.0 ** -23
        x_o, _ = rs.sample(np.full(u.size, chi), u, ur)
        got.append(x_o[x_o * g >= 2.0])
    xo = np.sort(np.concatenate(got)[:want])
    allv = np.concatenate([xi, xo])
    cdf_g = np.searchsorted(xi, allv, side="right") / m
    cdf_o = np.searchsorted(xo, allv, side="right") / want
    ks2 = np.max(np.abs(cdf_g - cdf_o))
    print(f"photons {m}  KS(exact) {ks1:.2e}  KS(oracle sampler) {ks2:.2e}")
    assert ks1 < 2e-3 and ks2 < 2e-3


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_pairs_one_step_parity(pair_table, dtype):
    """Photons with chi_ph log-uniform in [1e-2, 1e2] in per-particle fields: pair
    decisions, electron/positron records (rank order, ids, momenta, optical depth),
    dead photons and surviving optical depths against the oracle."""
    torch, q = need_gpu()
    n = 200000
    ph_in = workloads.pair_photons(n, seed=2)
    ph_in["k"] = ph_in["khat"] * (ph_in["chi_target"] /
                                  spectra.chi_photon(ph_in["khat"], ph_in["E"], ph_in["B"]))[:, None]
    tau = mc.init_tau(ph_in["id"], seed=2) * 0.05      # many events in one step
    cast = (lambda a: a.astype(np.float32).astype(np.float64)) if dtype == "f32" else (lambda a: a)
    k = cast(ph_in["k"])
    E, B = cast(ph_in["E"]), cast(ph_in["B"])
    ctx = q.Context(seed=2, kmax=4, flags=q.QED_FLAG_STATIC_PHOTONS)
    ctx.qed_build_tables(q.QED_FORMULA_I)
    ph = q.Species(n, dtype)
    el = q.Species(n + 10, dtype)
    po = q.Species(n + 10, dtype)
    ph.load(ph_in["x"], k, tau, ph_in["id"])
    ctx.qed_set_next_id(n)
    tdt = torch.float32 if dtype == "f32" else torch.float64
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda", torch.float32)
    fld = q.Fields(q.QED_FIELD_PER_PARTICLE, E=[dev(E[:, c]) for c in range(3)],
                   B=[dev(B[:, c]) for c in range(3)])
    dt = 0.01
    ctx.qed_create_pairs(fld, ph, el, po, dt, 3)
    st, rc = ctx.qed_get_status()
    ps = mc.PairSampler(pair_table, "f64" if dtype == "f64" else "q16")
    E32 = E.astype(np.float32).astype(np.float64)
    B32 = B.astype(np.float32).astype(np.float64)
    r = mc.photon_step(ph_in["x"], k, tau, ph_in["id"], E32, B32, dt=dt, step=3, seed=2,
                       sampler=ps, next_id=n, move=False)
    g_ph, g_el, g_po = ph.to_numpy(), el.to_numpy(), po.to_numpy()
    assert st["pairs"] == r["pairs"].size and st["scan_timeouts"] == 0 and st["dropped"] == 0
    np.testing.assert_array_equal(g_ph["id"], r["id"])
    np.testing.assert_array_equal(g_el["id"], r["electrons"]["id"])
    np.testing.assert_array_equal(g_po["id"], r["positrons"]["id"])
    rt = 1e-10 if dtype == "f64" else 3e-3
    for g, o in ((g_el, r["electrons"]), (g_po, r["positrons"])):
        ge = np.sqrt(1 + np.sum(g["p"] ** 2, axis=1))
        go = np.sqrt(1 + np.sum(o["p"] ** 2, axis=1))
        np.testing.assert_allclose(ge, go, rtol=rt)
        np.testing.assert_allclose(g["tau"], o["tau"], rtol=1e-12)
    alive = r["id"] != mc.DEAD_ID
    W = r["W"]
    np.testing.assert_allclose(g_ph["tau"][alive], r["tau"][alive], rtol=1e-9 if dtype == "f64" else 1e-4,
                               atol=(1e-9 if dtype == "f64" else 1e-4) * (W * dt).max())
    # compaction removes exactly the converted photons, in order
    ctx.qed_compact(ph)
    np.testing.assert_array_equal(ph.to_numpy()["id"], r["id"][alive])


def test_pair_spectrum_and_yield_1e7(pair_table):
    """1e7 photons at chi_ph = 1 (gamma_ph = 1000): pair yield in one step against
    1 - exp(-W dt) with W from the oracle quadrature (binomial z-test), and the
    electron energy fraction against the exact Eq. (6) CDF (one-sample KS) and the
    oracle's table sampler (two-sample KS), float32 path."""
    torch, q = need_gpu()
    n, gph, chi = 10_000_000, 1000.0, 1.0
    ctx = q.Context(seed=31, kmax=4, flags=q.QED_FLAG_STATIC_PHOTONS)
    ctx.qed_build_tables(q.QED_FORMULA_I)
    ph = q.Species(n, "f32")
    el = q.Species(n, "f32")
    po = q.Species(n, "f32")
    # photons along +x in B = b z: chi_ph = gamma_ph b / E_S
    b = chi * E_S / gph
    ph.load(np.zeros((n, 3)), np.tile([gph, 0.0, 0.0], (n, 1)), ids=np.arange(n, dtype=np.uint64))
    ctx.qed_init_optical_depth(ph, 0)
    ctx.qed_set_next_id(n)
    fld = q.Fields(q.QED_FIELD_UNIFORM, B=(0, 0, b))
    row = tables.fine_row("pair", chi, tables.PAIR_M)
    from oracle.constants import RATE_UNIT
    W = RATE_UNIT * 2 * row.total / gph
    dt = 1.0 / W                                   # P(pair) = 1 - e^-1
    ctx.qed_create_pairs(fld, ph, el, po, dt, 0)
    st, rc = ctx.qed_get_status()
    m = el.n()
    pr = 1 - math.exp(-W * dt)
    z = (m - n * pr) / math.sqrt(n * pr * (1 - pr))
    assert abs(z) < 4, z
    ge = torch.sqrt(1 + el.px[:m].double() ** 2 + el.py[:m].double() ** 2 + el.pz[:m].double() ** 2)
    xi = np.sort((ge / gph).cpu().numpy())
    # exact CDF of the full (symmetric) spectrum from the half-spectrum CDF
    P = row.F / row.total
    s_samp = np.log(xi) - np.log1p(-xi)
    Ph = np.interp(-np.abs(s_samp), row.s, P)          # half CDF at min(xi, 1-xi)
    Pe = np.where(s_samp <= 0, 0.5 * Ph, 1 - 0.5 * Ph)
    ks1 = max(np.max(np.arange(1, m + 1) / m - Pe), np.max(Pe - np.arange(m) / m))
    rng = np.random.default_rng(5)
    ps = mc.PairSampler(pair_table, "q16")
    u = (np.floor(rng.uniform(size=m) * 2 ** 23) + 0.5) * 2.0 ** -23
    ur = (np.floor(rng.uniform(size=m) * 2 ** 23) + 0.5) * 2.0 ** -23
    xh, omh = ps.sample_half(np.full(m, chi), u, ur)
    flip = rng.uniform(size=m) < 0.5
    xo = np.sort(np.where(flip, omh, xh))
    allv = np.concatenate([xi, xo])
    ks2 = np.max(np.abs(np.searchsorted(xi, allv, side="right") / m - np.searchsorted(xo, allv, side="right") / m))
    print(f"pairs {m} (z = {z:.2f})  KS(exact) {ks1:.2e}  KS(oracle sampler) {ks2:.2e}")
    assert ks1 < 2e-3 and ks2 < 2e-3


def _morton3(bx, by, bz, bits):
    """Morton code with x in the lowest bit of each triple (bit loop)."""
    code = np.zeros_like(bx)
    for k in range(bits):
        code |= ((bx >> k) & 1) << (3 * k)
        code |= ((by >> k) & 1) << (3 * k + 1)
        code |= ((bz >> k) & 1) << (3 * k + 2)
    return code


def test_sort_by_cell_stable_permutation():
    """qed_sort_by_cell: destination = source permuted by a stable sort of the
    nearest-node cell key (4x4x4 blocks along the Morton curve of their
    coordinates, cells z-major inside a block); counts and every array travel
    together."""
    torch, q = need_gpu()
    ctx = q.Context()
    n, cap, ng, L = 100003, 120000, 30, workloads.BOX_L
    rng = np.random.default_rng(9)
    x = rng.uniform(0, L, (n, 3)).astype(np.float32).astype(np.float64)
    x[:50] = x[50:100]              # repeated cells exercise stability
    p = rng.normal(size=(n, 3))
    tau = rng.uniform(size=n)
    ids = rng.permutation(n).astype(np.uint64)
    a, b = q.Species(cap, "f32"), q.Species(cap, "f32")
    a.load(x, p, tau, ids)
    grid = torch.zeros(ng ** 3 * 6, dtype=torch.float32, device="cuda")
    fld = q.Fields(q.QED_FIELD_GRID, grid=grid, n=ng, L=L)
    ctx.qed_sort_by_cell(fld, a, b)
    got = b.to_numpy()
    d = L / ng
    j = np.floor(x / d + 0.5).astype(np.int64)
    j[j >= ng] -= ng
    nb = (ng + 3) // 4
    mbits = int(np.ceil(np.log2(nb)))
    blk = _morton3(j[:, 0] // 4, j[:, 1] // 4, j[:, 2] // 4, mbits)
    key = blk * 64 + ((j[:, 2] % 4) * 4 + j[:, 1] % 4) * 4 + j[:, 0] % 4
    order = np.argsort(key, kind="stable")
    assert b.n() == n
    np.testing.assert_array_equal(got["id"], ids[order])
    np.testing.assert_array_equal(got["x"], x[order])
    np.testing.assert_array_equal(got["tau"], tau[order])


def test_method1_substep_f64_parity(rad_table_I):
    """The paper's method I with adaptive sub-steps (QED_FLAG_METHOD_I), float64,
    three Fig. 1 ensembles at dt = 0.03 (W dt = 0.06 / 0.45 / 0.27, i.e. 1, 3 and
    2 sub-steps): momenta, positions and photon lists against the oracle."""
    torch, q = need_gpu()
    ctx = q.Context(seed=5, kmax=4, flags=q.QED_FLAG_METHOD_I)
    ctx.qed_build_tables(q.QED_FORMULA_I)
    rad = mc.RadSampler(rad_table_I, "f64")
    dt, steps = 0.03, 10
    for k, e in enumerate(workloads.uniform_b_ensembles(2000, seed=5)):
        n = e["id"].size
        lep = q.Species(n, "f64")
        ph = q.Species(n * 4 * steps + 16, "f64")
        lep.load(e["x"], e["p"], np.zeros(n), e["id"])
        nid = 10**6 * (k + 1)
        ctx.qed_set_next_id(nid)
        fld = q.Fields(q.QED_FIELD_UNIFORM, B=(0, 0, e["b0"]))
        E = np.zeros((n, 3))
        B = np.tile([0.0, 0.0, e["b0"]], (n, 1))
        ox, op = e["x"].copy(), e["p"].copy()
        ids_ph = []
        for s in range(steps):
            ctx.qed_gather_push(fld, lep, -1, dt, s)
            ctx.qed_emit_photons(lep, ph, s)
            r = mc.lepton_step_method1_full(ox, op, e["id"], E, B, q=-1.0, dt=dt, step=s, seed=5,
                                            sampler=rad, next_id=nid)
            ox, op, nid = r["x"], r["p"], r["next_id"]
            ids_ph.append(r["photons"]["id"])
            gam_ref = r["photons"]["gamma"]
        st, rc = ctx.qed_get_status()
        g = lep.to_numpy()
        np.testing.assert_allclose(g["p"], op, rtol=1e-11, atol=1e-9)
        gph = ph.to_numpy()
        np.testing.assert_array_equal(gph["id"], np.concatenate(ids_ph))
        assert ctx.qed_get_next_id() == nid


def test_method1_dt_study():
    """The paper's time-step study (Fig. 3 discussion) with method I, float32, no
    recoil, chi ~ 1: Dt = 0.007/W, 0.2/W and 6/W with adaptive sub-steps reproduce
    the rate W (at 0.007/W and 0.2/W a single sub-step, as the paper finds the two
    alike); Dt = 6/W without sub-steps saturates at one event per step."""
    torch, q = need_gpu()
    from oracle.constants import RATE_UNIT
    n, b0, g = 200000, 2000.0, 206.0
    chi = g * math.sqrt(1 - 1 / g ** 2) * b0 / E_S
    W = RATE_UNIT * tables.fine_row("I", chi, tables.RAD_M, need_rho=False).total / g
    ens = workloads.uniform_b_ensembles(n, seed=8, triples=((b0, g),))[0]
    fld = q.Fields(q.QED_FIELD_UNIFORM, B=(0, 0, b0))
    for wdt, flags in ((0.007, 0), (0.2, 0), (6.0, 0), (6.0, q.QED_FLAG_NO_SUBSTEP)):
        ctx = q.Context(seed=8, kmax=4 if wdt < 1 else 4, flags=q.QED_FLAG_METHOD_I | q.QED_FLAG_NO_RECOIL | flags)
        ctx.qed_build_tables(q.QED_FORMULA_I)
        lep = q.Species(n, "f32")
        ph = q.Species(n * 4 * 3 + 16, "f32")
        lep.load(ens["x"], ens["p"], ids=ens["id"])
        ctx.qed_set_next_id(n)
        dt = wdt / W
        steps = 3
        for s in range(steps):
            ctx.qed_gather_push(fld, lep, -1, dt, s)
            ctx.qed_emit_photons(lep, ph, s)
        st, rc = ctx.qed_get_status()
        rate = st["events"] / (n * steps * dt)
        if flags:
            assert st["events"] == n * steps            # one event per step: rate 1/Dt = W/6
            assert abs(rate * dt - 1) < 1e-12
        elif wdt < 1:
            mean = n * steps * wdt
            print(f"method I, Dt = {wdt}/W: events {st['events']} (mean {mean:.0f})")
            assert abs(st["events"] - mean) < 4 * math.sqrt(mean)
        else:
            # 30 sub-steps of p = 0.2, kmax = 4 caps the events: compare the capped
            # binomial mean instead
            from math import comb
            N, pp = 30, wdt / 30
            pk = [comb(N, k) * pp ** k * (1 - pp) ** (N - k) for k in range(4)]
            mean1 = sum(k * pk[k] for k in range(4)) + 4 * (1 - sum(pk))
            assert abs(st["events"] / (n * steps) - mean1) < 0.01 * mean1


def test_box_staging_equals_global_gather():
    """The lepton pass's kernels and gathers give the same particles bit for bit.
    A float32 species on a grid takes two particles per thread when its capacity
    holds at least 64 particles per cell, one otherwise; in either, the
    workgroups of a cell-sorted dense species stage their stencil boxes in LDS
    (box_fallback near 0), those of the same particles in random order find
    their boxes too large and gather from global memory (box_fallback > 0).  The
    pushed momenta, positions and optical depths, matched by id, and the photons
    of the emission that follows are identical for the two orders; between the
    two kernels (separate compilations) they agree to float32 rounding.  2e6
    electrons on a 32^3 grid (61 per cell), standing wave a0 = 500, capacity 2e6
    (one particle per thread) or 2.2e6 (two): several XCD chunks of tiles and a
    ragged last tile."""
    torch, q = need_gpu()
    n, ng, L, dt, a0 = 2_000_003, 32, workloads.BOX_L, 0.01, 500.0
    ens = workloads.standing_wave_electrons(n, seed=12)
    x, p, ids = ens["x"], ens["p"], ens["id"]
    tau = mc.init_tau(ids, seed=3)
    tau[::7] *= 1e-3                                # some emitters within the step
    grid = torch.empty(ng ** 3 * 6, dtype=torch.float32, device="cuda")
    fld = q.Fields(q.QED_FIELD_GRID, grid=grid, n=ng, L=L)
    res = {}
    for cap in (n, 2_200_000):
        for name in ("sorted", "random"):
            print(f"lepton pass: capacity {cap}, {name} order", flush=True)
            ctx = q.Context(seed=3, kmax=4)
            ctx.qed_build_tables(q.QED_FORMULA_I)
            ctx.qed_fill_standing_wave(grid, ng, L, a0, 0.21)
            a = q.Species(cap, "f32")
            if name == "sorted":
                src = q.Species(cap, "f32")
                src.load(x, p, tau, ids)
                ctx.qed_sort_by_cell(fld, src, a)
                del src
            else:
                perm = np.random.default_rng(5).permutation(n)
                a.load(x[perm], p[perm], tau[perm], ids[perm])
            ph = q.Species(400_000, "f32")
            ctx.qed_set_next_id(n)
            ctx.qed_reserve(cap)
            ctx.qed_get_status(check=False)
            ctx.qed_gather_push(fld, a, -1, dt, 0)
            st, _ = ctx.qed_get_status()
            g = a.to_numpy()
            o = np.argsort(g["id"])
            out = {k: g[k][o] for k in ("x", "p", "tau", "id")}
            ctx.qed_emit_photons(a, ph, 0)
            st2, _ = ctx.qed_get_status()
            gp = ph.to_numpy()
            # photon ids follow the emitters' storage order: compare the photons
            # as a set, ordered by their emitter's position, energy and time
            key = np.lexsort((gp["tau"], gp["p"][:, 0], gp["x"][:, 2], gp["x"][:, 1], gp["x"][:, 0]))
            out.update(ph_x=gp["x"][key], ph_k=gp["p"][key], ph_tau=gp["tau"][key])
            res[cap, name] = (st, st2, out)
            ctx.close()
    for (cap, name), (st, st2, out) in res.items():
        print(f"capacity {cap}, {name}: box fallbacks {st['box_fallback']}, photons {out['ph_x'].shape[0]}")
    for cap in (n, 2_200_000):
        (s0, e0, r0), (s1, e1, r1) = res[cap, "sorted"], res[cap, "random"]
        assert r0["ph_x"].shape[0] > 1000 and e0["dropped"] == 0 and e1["dropped"] == 0
        # within one kernel the two gathers agree bit for bit
        for k in r0:
            np.testing.assert_array_equal(r1[k], r0[k])
        # (a sorted tile can straddle two distant blocks and fall back too: rare)
        assert s1["box_fallback"] > 0 and s0["box_fallback"] * 100 < s1["box_fallback"]
    # the two kernels are separate compilations whose fused multiply-adds
    # differ: the particles agree to float32 rounding (positions within 2 ulp of
    # the box length 2 pi, momenta within 16 ulp of the larger of |p| and the
    # step's kick a0 dt, the magnitude of the push's intermediates), the photons
    # in number and energy
    a, b = res[n, "sorted"][2], res[2_200_000, "sorted"][2]
    np.testing.assert_array_equal(a["id"], b["id"])
    for k, scale, tol in (("x", 1.0, 2.0 ** -20), ("p", np.maximum(np.abs(a["p"]), a0 * dt), 2.0 ** -19)):
        d = np.max(np.abs(b[k] - a[k]) / scale)
        print(f"one vs two particles per thread: {k} max diff {d:.2e}, "
              f"{np.mean(b[k] != a[k]):.2e} of the values differ")
        assert d <= tol
    # the optical depth drops by W dt <~ 0.1, W within ~1e-6 (chi from the momenta above)
    np.testing.assert_allclose(b["tau"], a["tau"], rtol=1e-6, atol=1e-6)
    assert abs(b["ph_x"].shape[0] - a["ph_x"].shape[0]) <= 2
    ga = np.sort(np.linalg.norm(a["ph_k"], axis=1))
    gb = np.sort(np.linalg.norm(b["ph_k"], axis=1))
    if ga.size == gb.size:
        np.testing.assert_allclose(gb, ga, rtol=1e-5)


@pytest.mark.parametrize("n", [1, 255, 257, (1 << 20) - 1, 1 << 20, (1 << 20) + 77])
def test_sample_edges(rad_table_I, pair_table, n):
    """Both kernels of the sampler over chi and gamma of every branch: zero, below
    and above the tables, where float32 loses h_pair, gamma below 2.  ln W is float32
    of a sum of terms up to 300 whose tables are float32 (2e-5 relative in W and four
    units in the last place of ln W); where h_pair is subnormal in float32, one unit
    of it more (half below one unit either way: -inf)."""
    torch, q = need_gpu()
    ctx = q.Context(seed=6)
    ctx.qed_build_tables(q.QED_FORMULA_I)
    edge = np.array([0.0, 1e-30, 1e-6, 9.99e-4, 1e-3, 0.00999, 0.01, 0.011, 0.02, 0.0255, 0.026, 0.03, 0.0306, 0.031,
                     1.0, 99.9, 100.0, 101.0, 1e6])
    chi = np.resize(edge, n)
    gam = np.resize(np.array([1.0, 1.999, 2.0, 2.5, 1e3, 1e7, 1e-3]), n)
    ids = np.arange(n, dtype=np.uint64) * np.uint64(0x9E3779B97F4A7C15)
    dev = lambda a, dt: torch.from_numpy(a).to("cuda", dt)
    tchi, tg = dev(chi, torch.float64), dev(gam, torch.float64)
    tid = dev(ids.view(np.int64), torch.int64)
    from oracle import philox
    u = philox.uniform(philox.stream(ids, 6, 3, philox.LEPTON_EVENT, 0))
    rad, pair = mc.RadSampler(rad_table_I, "f64"), mc.PairSampler(pair_table, "f64")
    with np.errstate(divide="ignore"):
        lw, lwp = np.log(rad.rate(chi, gam)), np.log(pair.rate(chi, gam))
    h = pair.rate(chi, np.full(n, 2.0)) * 2.0 / RATE_UNIT
    # float32 rounds the mixing fraction of a row by up to 1e-5: not the draws beside it
    with np.errstate(divide="ignore"):
        pos = np.log(np.maximum(chi, tables.RAD_CHI_MIN) / tables.RAD_CHI_MIN) / np.log(100.0 / tables.RAD_CHI_MIN) * 255
    beside = np.abs((pos - u[:, 2] + 0.5) % 1.0 - 0.5) < 1e-4
    for prec, storage, tol_s in ((q.QED_F64, "f64", 1e-10), (q.QED_F32, "q16", 3e-3)):
        print(f"sample: n={n} precision {prec}", flush=True)
        lnw = torch.empty(n, dtype=torch.float32, device="cuda")
        xi, lnwp = torch.empty_like(lnw), torch.empty_like(lnw)
        ctx.qed_sample(tchi, tg, tid, prec, 3, lnw, xi, lnwp)
        got = [v.cpu().numpy().astype(np.float64) for v in (lnw, xi, lnwp)]
        near = lambda a, b, more: np.all((a == b) | (np.abs(a - b) <= 2e-5 + 4 * 2.0 ** -23 * np.abs(b) + more))
        with np.errstate(invalid="ignore"):
            assert near(got[0], lw, 0.0)
            if prec == q.QED_F64:
                ok = np.ones(n, bool)
                assert near(got[2], lwp, 0.0)
            else:
                unit32 = 2.0 ** -149
                ok = h > 4 * unit32
                assert near(got[2][ok], lwp[ok], unit32 / np.maximum(h[ok], 2.0 ** -126) + 2 * unit32 / h[ok])
                assert np.all(np.isneginf(got[2][h < 0.25 * unit32]))
        xr, _ = mc.RadSampler(rad_table_I, storage).sample(chi, u[:, 0], u[:, 2])
        far = np.abs(got[1] - xr) > tol_s * xr * (1 - xr) + 4e-7 * xr + 2.0 ** -149
        assert not np.any(far & ~beside)
    ctx.close()
