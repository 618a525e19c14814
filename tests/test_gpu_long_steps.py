"""Long steps of eccentric orbits (e 0.6 to 0.99, 0.1 to 6 rad of mean anomaly
a step) on the GPU: every kernel that goes from one solved instant to the next
holds the exact position at the next one.

Boxes against the oracle's within 1e-9 relative, as for short steps (the two
sides differ by rounding only).  Witnesses against positions from a bisection of
Kepler's equation; M of some 25 rad is rounded to 4e-15, which 1 - e cos E >= 0.01
and a = 20 000 km make 1e-8 km at most, so a distance within 1e-6 km of the
threshold may go either way.  Refined leaves as in the refinement's own tests:
boxes that touch to within 1e-5 km may go either way.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_1901_10475_amd as cd
from tests.gpu_util import assert_boxes_close, gpu_to_object_major, need_gpu, say

pytestmark = pytest.mark.gpu
MU, TICK = oracle.MU_EARTH, 1e-3
RULES = [cd.CD_BOX_SPEED, cd.CD_BOX_INTERVAL_NU, cd.CD_BOX_INTERVAL_E]


def _orbits(rng, n, a, e):
    return np.column_stack([np.broadcast_to(a, n), e, rng.uniform(0, np.pi, n),
                            rng.uniform(0, 2 * np.pi, (n, 3))])


def _ticks(dM, a):
    return np.maximum(np.rint(dM / np.sqrt(MU / a ** 3) / TICK), 1).astype(np.uint32)


def _positions(el, t_s):
    """[n, len(t_s), 3], Kepler's equation by bisection."""
    a, e, inc, raan, argp, m0 = (el[:, k, None] for k in range(6))
    M = m0 + np.sqrt(MU / a ** 3) * t_s[None, :]
    lo, hi = M - e, M + e
    for _ in range(60):
        mid = 0.5 * (lo + hi)
        up = (mid - M) - e * np.sin(mid) > 0
        lo, hi = np.where(up, lo, mid), np.where(up, mid, hi)
    E = 0.5 * (lo + hi)
    u, v = a * (np.cos(E) - e), a * np.sqrt(1 - e * e) * np.sin(E)
    cO, sO, ci, si, cw, sw = (f(x) for x in (raan, inc, argp) for f in (np.cos, np.sin))
    P = (cO * cw - sO * sw * ci, sO * cw + cO * sw * ci, sw * si)
    Q = (-cO * sw - sO * cw * ci, -sO * sw + cO * cw * ci, cw * si)
    return np.stack([u * p + v * q for p, q in zip(P, Q)], axis=2)


@pytest.mark.parametrize("layout", [cd.CD_LAYOUT_OBJECT, cd.CD_LAYOUT_SORTED])
@pytest.mark.parametrize("rule", RULES)
@pytest.mark.parametrize("dM", [0.1, 0.5, 1.5, 3.0, 6.0])
def test_uniform_boxes(dM, rule, layout):
    need_gpu()
    say("long uniform steps, dM", dM, "rule", rule, "layout", layout)
    n, K = 3000, 8
    rng = np.random.default_rng(int(10 * dM))
    el = _orbits(rng, n, 20_000.0, np.resize([0.6, 0.65, 0.75, 0.85, 0.9, 0.95, 0.97], n))
    dt = int(_ticks(dM, 20_000.0))
    T = K * dt - 337
    p = cd.params_struct(TICK, MU, 1.0, T, dt, box_rule=rule)
    bp = cd.BroadPhase(n, p, None, layout=layout, in_tree=layout == cd.CD_LAYOUT_SORTED)
    cd.cd_build_boxes(cd.soa(el), None, p, bp.boxes, bp.ws_boxes)
    lo, hi, t0, t1, obj = bp.boxes.to_host()
    g = gpu_to_object_major(obj, n, K)
    ob = oracle.boxes(el, dt, T, TICK, 1.0, rule=rule)
    assert np.array_equal(t0[g], ob.t0) and np.array_equal(t1[g], ob.t1)
    assert_boxes_close(lo[g], hi[g], ob.lo, ob.hi, el[ob.obj, 0])


@pytest.mark.parametrize("rule", RULES)
def test_per_object_boxes(rule):
    need_gpu()
    say("long per-object steps, rule", rule)
    n, T = 6000, 100_000_000
    rng = np.random.default_rng(5)
    a = rng.uniform(12_000, 40_000, n)
    el = _orbits(rng, n, a, rng.uniform(0.6, 0.97, n))
    dt = _ticks(np.exp(rng.uniform(np.log(0.1), np.log(6.0), n)), a)
    p = cd.params_struct(TICK, MU, 1.0, T, 0, box_rule=rule)
    bp = cd.BroadPhase(n, p, torch.from_numpy(dt.view(np.int32)).cuda())
    cd.cd_build_boxes(cd.soa(el), bp.dt, p, bp.boxes, bp.ws_boxes)
    lo, hi, t0, t1, obj = bp.boxes.to_host()
    ob = oracle.boxes(el, dt, T, TICK, 1.0, rule=rule)
    assert np.array_equal(obj, ob.obj) and np.array_equal(t0, ob.t0) and np.array_equal(t1, ob.t1)
    assert_boxes_close(lo, hi, ob.lo, ob.hi, el[ob.obj, 0])


def _windows(rng, n, K, D, pairs):
    """Records of two instants, k D and (k + 1) D, for every pair and k < K."""
    k = np.tile(np.arange(K, dtype=np.int64), len(pairs))
    ij = np.repeat(pairs, K, axis=0)
    return np.column_stack([ij, k * D, (k + 1) * D + 1]).astype(np.uint32)


def test_first_witness():
    """Neighbours on one orbit, whose distance shrinks as they leave perigee."""
    need_gpu()
    say("first witness over 0.24 rad")
    n, K, thr = 4000, 60, 50.0
    rng = np.random.default_rng(7)
    el = _orbits(rng, n, 20_000.0, np.repeat(rng.uniform(0.93, 0.99, n // 2), 2))
    el[1::2] = el[::2]
    el[1::2, 5] += thr / 20_000.0 * np.exp(rng.uniform(np.log(0.1), np.log(3.0), n // 2))
    D = int(_ticks(0.24, 20_000.0))
    T = K * D
    rec = _windows(rng, n, K, D, np.arange(n).reshape(-1, 2))
    p = cd.params_struct(TICK, MU, thr, T, D)
    wit, _ = cd.cd_first_witness(cd.soa(el), p, D, torch.from_numpy(rec.view(np.int32)).cuda())
    got = wit.cpu().numpy().view(np.uint32).reshape(n // 2, K)
    P = _positions(el, np.arange(K + 1) * D * TICK)
    d = np.abs(P[::2] - P[1::2]).max(axis=2)
    now, then = d[:, :-1] <= thr, d[:, 1:] <= thr
    k = np.arange(K)[None, :]
    want = np.where(now, k * D, np.where(then, (k + 1) * D, cd.CD_NO_WITNESS))
    clear = np.abs(d - thr) > 1e-6
    sure = clear[:, :-1] & clear[:, 1:]
    assert (~now & then & sure).sum() > 500
    assert np.array_equal(got[sure], want[sure].astype(np.uint32))


@pytest.mark.parametrize("rule", [cd.CD_BOX_SPEED, cd.CD_BOX_INTERVAL_E])
def test_refined_spans(rule):
    """Spans of two instants, each kept where the two objects' boxes meet."""
    need_gpu()
    say("refinement over 0.24 rad, rule", rule)
    n, K = 2000, 40
    rng = np.random.default_rng(9)
    el = _orbits(rng, n, 20_000.0, rng.uniform(0.93, 0.99, n))
    D = int(_ticks(0.24, 20_000.0))
    T = K * D
    i = rng.integers(0, n - 1, 5000)
    pairs = np.unique(np.column_stack([i, i + 1 + rng.integers(0, n, 5000) % (n - 1 - i)]), axis=0)
    rec = _windows(rng, n, K, D, pairs)
    p = cd.params_struct(TICK, MU, 1.0, T, D, box_rule=rule)
    got = cd.cd_refine_records(cd.soa(el), p, D, torch.from_numpy(rec.view(np.int32)).cuda(),
                               min_steps=2).cpu().numpy().view(np.uint32)
    want = oracle.refine(el, rec, T, TICK, 1.0, D, 2, rule=rule)
    assert 100 < len(want) < len(rec)
    for i, j, a, b in {tuple(x) for x in got.tolist()} ^ {tuple(x) for x in want.tolist()}:
        ta, tb = a * TICK, (b - 1) * TICK
        if rule == cd.CD_BOX_SPEED:
            box = []
            for o in (i, j):
                pa, pb = oracle.position(el[o], ta), oracle.position(el[o], tb)
                grow = oracle.vmax(*el[o, :2]) * (tb - ta) / 2 + 0.5
                box.append((np.minimum(pa, pb) - grow, np.maximum(pa, pb) + grow))
        else:
            box = [oracle.box_interval(el[o], ta, tb, 1.0, rule) for o in (i, j)]
        (li, hi), (lj, hj) = box
        assert abs(np.max(np.maximum(li - hj, lj - hi))) <= 1e-5, (i, j, a, b)
