"""One species' arrays through descriptors of different capacity: the push and the
emission that follows it need not be given the same one, as long as both hold the
particles present.  The photons are those of a push and an emission with one
descriptor: the same kernels on the same particles, so ids, counts and order are
equal and values agree to the roundings of the two compilations of an event that a
capacity chooses between (64 units in the last place)."""
import copy

import numpy as np
import pytest

from tests.gpu_helpers import need_gpu

import workloads

pytestmark = pytest.mark.gpu

ULPS = {"f32": 64 * 2.0 ** -24, "f64": 64 * 2.0 ** -53}


def _with_capacity(sp, capacity):
    """The same arrays with `capacity` slots in the descriptor."""
    v = copy.copy(sp)
    v.c = type(sp.c).from_buffer_copy(sp.c)
    v.c.capacity = v.capacity = capacity
    return v


def _context(q, surrogate):
    ctx = q.Context(seed=9, kmax=4, flags=q.QED_FLAG_SURROGATE if surrogate else 0)
    ctx.qed_build_tables(q.QED_FORMULA_I)
    if surrogate:                       # (weights of any kind: a rate outside the envelope takes the table)
        for net in (0, 1):
            m = q.lib().qed_surrogate_params(net)
            ctx.qed_surrogate_io(net, np.random.default_rng(net).normal(0, 0.05, m).astype(np.float32))
    return ctx


def _electrons(q, ctx, n, capacity, dtype):
    ens = workloads.uniform_b_ensembles(n, seed=5, triples=((2000.0, 206.0),))[0]
    lep = q.Species(capacity, dtype)
    lep.load(ens["x"], ens["p"], np.zeros(n), ens["id"])
    ctx.qed_init_optical_depth(lep, 0)
    ctx.qed_set_next_id(n)
    return lep


def _same(a, b, dtype):
    for u, v in zip(a[:2], b[:2]):
        assert np.array_equal(u["id"], v["id"])
        scale = np.maximum(np.abs(v["p"]), np.abs(v["p"]).max(axis=1, keepdims=True))
        assert np.all(np.abs(u["p"] - v["p"]) <= ULPS[dtype] * scale)
        assert np.all(np.abs(u["tau"] - v["tau"]) <= ULPS[dtype] * np.maximum(1.0, np.abs(v["tau"])))
    assert a[2] == b[2]


@pytest.mark.parametrize("dtype,surrogate", [("f32", False), ("f64", False), ("f32", True)])
def test_emission_with_more_slots_than_the_push_reserved(dtype, surrogate):
    """Only the push reserves the context; the emission takes up to twice its slots."""
    torch, q = need_gpu()
    n, push, emit = 50_000, 1_100_000, 2_200_000
    fld = q.Fields(q.QED_FIELD_UNIFORM, B=(0, 0, 2000.0))
    out = []
    for caps in ((push, emit), (emit, emit)):
        print(f"emission: {dtype} surrogate={surrogate} slots {caps}", flush=True)
        ctx = _context(q, surrogate)
        lep, ph = _electrons(q, ctx, n, emit, dtype), q.Species(6 * n, dtype)
        for s in range(2):
            ctx.qed_gather_push(fld, _with_capacity(lep, caps[0]), -1, 0.02, s)
            ctx.qed_emit_photons(_with_capacity(lep, caps[1]), ph, s)
        out.append((ph.to_numpy(), lep.to_numpy(), ctx.qed_get_status()[0]))
        ctx.close()
    assert out[0][2]["photons"] > 1000
    _same(out[0], out[1], dtype)


@pytest.mark.parametrize("dtype,surrogate", [("f32", False), ("f64", False), ("f32", True)])
@pytest.mark.parametrize("push,emit", [((1 << 17) + 1, 1 << 17), (1 << 17, (1 << 17) + 1), (1 << 17, 1 << 20)])
def test_emission_with_other_slots_than_the_push(dtype, surrogate, push, emit):
    """After calls that left the scan state of every tile behind: the capacity chooses
    the tiles (256 particles up to 2^17, else 512 emitters or more), so what the push
    clears for its own is not what the emission needs."""
    torch, q = need_gpu()
    n = 1 << 17
    fld = q.Fields(q.QED_FIELD_UNIFORM, B=(0, 0, 2000.0))
    out = []
    for caps in ((push, emit), (emit, emit)):
        print(f"emission: {dtype} surrogate={surrogate} slots {caps}", flush=True)
        ctx = _context(q, surrogate)
        lep, ph = _electrons(q, ctx, n, max(push, emit), dtype), q.Species(12 * n, dtype)
        for s, (a, b) in enumerate([(emit, emit), (push, push), caps, caps]):
            ctx.qed_gather_push(fld, _with_capacity(lep, a), -1, 0.02, s)
            ctx.qed_emit_photons(_with_capacity(lep, b), ph, s)
        out.append((ph.to_numpy(), lep.to_numpy(), ctx.qed_get_status()[0]))
        ctx.close()
    assert out[0][2]["photons"] > 10_000 and out[0][2]["dropped"] == 0
    _same(out[0], out[1], dtype)
