"""Direct Riemannian illumination (rt_illuminate) on the GPU.

Several geodesics may join a surface point to the light, so the GPU's
answer is checked for validity rather than against one reference solution:
the FP64 oracle integrates the returned geodesic and must land on the light,
recomputes the Lambert term in the metric from the returned direction, and
recomputes the visibility along it.  In flat space everything has a closed
form."""
import numpy as np
import pytest

import oracle
import workloads as W
from tests import exact

pytestmark = pytest.mark.gpu

LIGHT = dict(pos=(2.5, 3.5, -3.0), h=0.01, tol=1e-4, max_iters=16, max_steps=4000)


def say(*a):
    print("[gpu-case]", *a, flush=True)


@pytest.fixture(scope="module")
def rt():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2005_05386_amd import rt as _rt
    return _rt


def _run(rt, wl, light=LIGHT):
    tr = rt.Tracer(0)
    tr.set_metric(wl["metric"])
    tr.set_scene(wl["scene"])
    out = tr.trace(wl["camera"], wl["rule"])
    sh = tr.illuminate(wl["camera"], out, light)
    tr.sync()
    tra = rt.to_numpy(out)
    return tra, {k: v.cpu().numpy() for k, v in sh.items()}


def _grad_F(scene, oid, q):
    """Outward gradient of the implicit function of object oid at q (FP64)."""
    sp = np.asarray(scene["spheres"], np.float64).reshape(-1, 4)
    pl = np.asarray(scene["planes"], np.float64).reshape(-1, 4)
    to = np.asarray(scene["tori"], np.float64).reshape(-1, 8)
    if oid < len(sp):
        return 2.0 * (q - sp[oid, :3])
    oid -= len(sp)
    if oid < len(pl):
        return pl[oid, :3].copy()
    c, a, R = to[oid - len(pl), :3], to[oid - len(pl), 3:6], to[oid - len(pl), 6]
    x = q - c
    ax = x @ a
    rad = x - ax * a
    rn = np.linalg.norm(rad)
    e = rn - R
    return (e * rad / rn + ax * a) / np.hypot(e, ax)


def test_flat_space_closed_form(rt):
    """g = I: the geodesic to the light is the segment, found at once; the
    Lambert term is n . (L - q)/|L - q| and the visibility is the segment's."""
    say("illumination, flat space 64x48")
    wl = W.with_size(W.get("bumps16_1080p"), 64, 48)
    wl["metric"] = W.metric(W.EUCLID)
    tra, sh = _run(rt, wl)
    L = np.array(LIGHT["pos"], np.float64)
    hit = tra["id"] >= 0
    assert (sh["status"][~hit] == -3).all()
    assert (sh["status"][hit] >= 0).all(), np.unique(sh["status"][hit])
    n_bad = 0
    for p in np.nonzero(hit)[0]:
        q = tra["hit"][p].astype(np.float64)
        d = L - q
        T = np.linalg.norm(d)
        v = d / T
        assert np.abs(sh["dir"][p] - v).max() < 2e-5, (p, sh["dir"][p], v)
        assert abs(sh["len"][p] - T) < 1e-4 * max(1.0, T)
        gF = _grad_F(wl["scene"], tra["id"][p], q)
        cos = gF @ v / np.linalg.norm(gF)
        if cos <= 0:
            n_bad += sh["status"][p] != 2
            continue
        qs = q + 1e-3 * v
        t, oid = exact.line_hits(qs, v[None, :], wl["scene"], T - 1e-3)
        lit = oid[0] < 0
        if lit:
            n_bad += not (sh["status"][p] == 1 and abs(sh["shade"][p] - cos) < 1e-4)
        else:
            n_bad += sh["status"][p] != 0
    assert n_bad <= max(2, 0.002 * hit.sum()), (n_bad, hit.sum())


# found: the least fraction of hit pixels for which a geodesic is found
# (Newton from the straight segment, then retries from converged
# neighbours, then the continuation in the light position).  The quadric's
# slope grows linearly with the distance from the origin: on the way to the
# light many geodesics bend far from the segment, and it keeps the most
# pixels unsolved.
@pytest.mark.parametrize("name,w,h,found_min", [("bumps16_1080p", 64, 40, 0.99), ("twist_4k", 64, 40, 0.99),
                                                ("deform16_1080p", 48, 30, 0.99), ("rdeform16_1080p", 48, 30, 0.99),
                                                ("abumps16_1080p", 64, 40, 0.99),
                                                ("quadric_1080p", 64, 40, 0.9)])
def test_curved_geodesics_reach_the_light(rt, name, w, h, found_min):
    """Curved metrics: the oracle integrates each returned geodesic in FP64
    and lands on the light; the Lambert term and the visibility recomputed
    in FP64 from the returned direction agree."""
    say("illumination, %s %dx%d" % (name, w, h))
    wl = W.with_size(W.get(name), w, h)
    tra, sh = _run(rt, wl)
    _check_found(wl, tra, sh, found_min)


def test_illum_1080p_sampled(rt):
    """The benchmarked 1080p frame and launch configuration: the counts
    over every hit pixel, and the FP64 checks on a seeded sample of 400
    pixels that found a geodesic."""
    say("illumination, illum_1080p full frame, 400 sampled pixels")
    wl = W.get("illum_1080p")
    assert tuple(wl["light"]["pos"]) == LIGHT["pos"] and wl["light"]["h"] == LIGHT["h"]
    tra, sh = _run(rt, wl, light=wl["light"])
    _check_found(wl, tra, sh, 0.99, sample=400)


def _check_found(wl, tra, sh, found_min, sample=None):
    orc = oracle.Oracle(wl["metric"], wl["scene"])
    L = np.array(LIGHT["pos"], np.float64)
    hit = np.nonzero(tra["id"] >= 0)[0]
    st = sh["status"]
    assert (st[tra["id"] < 0] == -3).all()
    found = hit[st[hit] >= 0]
    say("hits %d found %d lit %d shadowed %d facing away %d" % (len(hit), len(found), (st == 1).sum(),
                                                                (st == 0).sum(), (st == 2).sum()))
    assert len(found) >= found_min * len(hit)
    check = found if sample is None else np.sort(np.random.default_rng(5).choice(found, sample, replace=False))
    worst_end = worst_cos = 0.0
    vis_bad = 0
    for p in check:
        q = tra["hit"][p].astype(np.float64)
        v = sh["dir"][p].astype(np.float64)
        g = orc.metric_tensor(q)
        v = v / np.sqrt(v @ g @ v)
        T = float(sh["len"][p])
        z, ok = orc.shoot(q, v, T, LIGHT["h"])
        assert ok
        worst_end = max(worst_end, np.abs(z[:3] - L).max())
        gF = _grad_F(wl["scene"], tra["id"][p], q)
        cos = gF @ v / np.sqrt(gF @ np.linalg.solve(g, gF))
        if st[p] == 2:
            assert cos < 1e-3, (p, cos)
            continue
        assert cos > -1e-3
        if st[p] == 1:
            worst_cos = max(worst_cos, abs(sh["shade"][p] - cos))
        clear = orc.geodesic_clear(q, v, T, LIGHT["h"], 1e-3)
        vis_bad += clear != (st[p] == 1)
    say("worst end %.2e, worst cos %.2e, visibility disagreements %d" % (worst_end, worst_cos, vis_bad))
    # end: the GPU stops once its FP32 shot lands within tol = 1e-4 (max
    # norm); the FP64 integration of the returned direction adds the FP32
    # trajectory's rounding drift (measured worst 1.30e-4, on the quadric)
    assert worst_end < 2e-4
    # Lambert term: FP32 assembly and inversion of g at q; the quadric's
    # steep slopes make g worst conditioned (measured worst 2.0e-5 there,
    # 3.8e-7 on the other metrics)
    assert worst_cos < 5e-5
    # visibility: none measured; one grazing geodesic may be decided
    # differently in FP32 and FP64
    assert vis_bad <= max(1, 0.0025 * len(check))


def test_multi_set_equals_single_sets(rt):
    """Three parameter sets in one call give, set by set, bitwise the
    single-set results (the single-set kernels read the bump table with
    scalar loads, the multi-set ones per lane)."""
    say("illumination, 3 parameter sets in one call vs one by one")
    wl = W.with_size(W.get("adjoint_64x512", n_sets=3), 40, 32)
    _, sh = _run(rt, wl)
    n = 40 * 32
    for s in range(3):
        one = dict(wl)
        one["metric"] = dict(wl["metric"], bumps=wl["metric"]["bumps"][s:s + 1])
        _, shs = _run(rt, one)
        say("set %d: %d lit" % (s, (shs["status"] == 1).sum()))
        for k in ("status", "shade", "dir", "len"):
            assert np.array_equal(sh[k][s * n:(s + 1) * n], shs[k]), (s, k)


def test_edge_cases(rt):
    """Empty pixel lists and tiny frames: a frame with no hit (all -3, no
    Newton work), a single pixel, and one Newton iteration only, where only
    pixels whose straight segment already lands within tol may be lit."""
    say("illumination edge cases")
    base = W.get("bumps16_1080p")
    # flat space, the camera looks up and away from every object (every ray
    # rises, the objects lie below and ahead): no hit, every list empty
    wl = W.with_size(base, 16, 8)
    wl["metric"] = W.metric(W.EUCLID)
    wl["camera"] = W.camera(16, 8, eye=(0.0, 0.0, -10.0), forward=(0.0, 1.0, 0.0), up=(0.0, 0.0, 1.0))
    tra, sh = _run(rt, wl)
    assert (tra["id"] < 0).all()
    assert (sh["status"] == -3).all() and (sh["shade"] == 0).all() and (sh["len"] == 0).all()
    # one pixel, aimed down at the plane y = -1 (or a sphere before it)
    wl = W.with_size(base, 1, 1)
    wl["camera"] = W.camera(1, 1, eye=(0.0, 0.0, -4.0), forward=(0.0, -0.5, 1.0))
    tra, sh = _run(rt, wl)
    assert tra["id"][0] >= 0 and sh["status"][0] in (-1, 0, 1, 2)
    # one iteration: a pixel is found only if its straight segment lands
    wl = W.with_size(base, 32, 20)
    tra, sh = _run(rt, wl, light=dict(LIGHT, max_iters=1))
    found = np.nonzero(sh["status"] >= 0)[0]
    orc = oracle.Oracle(wl["metric"], wl["scene"])
    L = np.array(LIGHT["pos"], np.float64)
    for p in found[:50]:
        q = tra["hit"][p].astype(np.float64)
        d = L - q
        v = d / np.sqrt(d @ orc.metric_tensor(q) @ d)
        assert np.abs(sh["dir"][p] / np.linalg.norm(sh["dir"][p]) - v / np.linalg.norm(v)).max() < 1e-5, p


@pytest.mark.parametrize("w,h", [(24, 16), (160, 104)])
@pytest.mark.parametrize("n", [1, 16, 17, 32])
def test_spread_bumps_equal_the_walk(rt, n, w, h):
    """Isotropic tables of up to 32 bumps end their Newton iterations with the
    bumps spread over the lanes of a wave (a table of up to 16, and of up to
    32; lists that start short and ones handed over); a longer table walks
    them.  Bumps of amplitude zero make the table long and add nothing, so the
    outputs are equal bit for bit."""
    say("illumination", w, h, "bumps", n, "against the same padded to 33")
    wl = W.with_size(W.get("bumps16_1080p"), w, h)
    rng = np.random.default_rng(n)
    b = np.concatenate([rng.uniform(0.1, 0.5, (n, 1)), rng.uniform(-2, 2, (n, 3)), rng.uniform(0.15, 0.4, (n, 1))], 1)
    pad = np.tile(np.array([[0.0, 3.0, 3.0, 3.0, 0.3]]), (33 - n, 1))
    res = []
    for bumps in (b, np.concatenate([b, pad])):
        metric = dict(wl["metric"], bumps=bumps[None].astype(np.float32))
        res.append(_run(rt, dict(wl, metric=metric)))
    (ta, sa), (tb, sb) = res
    assert np.array_equal(ta["hit"], tb["hit"]) and (ta["id"] >= 0).any()
    for k in sa:
        assert np.array_equal(sa[k], sb[k], equal_nan=True), k


@pytest.mark.parametrize("n", [4, 33])
def test_shot_off_unit_speed(rt, n):
    """A shot that leaves a bump faster than 1 (RK4 with h = 0.03 through the tip
    of a = 0.6, sigma = 0.1, the distance to it searched with the oracle)
    flies as far as its own speed allows, here to a sharp bump 25 units on
    (the last flight starts half way, where the tip is no nearer).  The
    same pixel with one more bump, of amplitude zero and a cut that holds the
    scene, flies nowhere: equal bit for bit, for bumps spread over the lanes and
    walked.  (The light is 280 units off, so that the first target of the
    continuation, an eighth of the way, lies behind that bump too.)"""
    say("illumination, shot off unit speed, %d bumps" % n)
    wl = W.with_size(W.get("bumps16_1080p"), 1, 1)
    wl["scene"] = W.scene(planes=[(0.0, 1.0, 0.0, -1.0)])
    wl["camera"] = W.camera(1, 1, eye=(0.0, 0.5, -4.0), forward=(0.0, -0.75, 1.0))
    light = dict(LIGHT, pos=(27.0, 280.0, 15.0), h=0.03, max_steps=20000)

    def run(bumps):
        b = np.concatenate([bumps, np.tile([[0.0, 40.0, -40.0, 40.0, 0.1]], (n - len(bumps), 1))])
        out = []
        for sigma in (0.1, 1000.0):
            b[-1, 4] = sigma
            out.append(_run(rt, dict(wl, metric=dict(wl["metric"], bumps=b[None].astype(np.float32))), light=light))
        return out
    q = run(np.zeros((0, 5)) + 0.1)[0][0]["hit"][0].astype(np.float64)
    e = np.array(light["pos"]) - q
    e /= np.linalg.norm(e)
    best = None
    for d in np.arange(0.75, 0.78, 0.001):
        tip = np.array([[0.6, *(q + d * e), 0.1]]).astype(np.float32)
        z, ok = oracle.Oracle(W.metric(W.GRAPH_GAUSS, bumps=tip), wl["scene"]).shoot(q, e, 3.0, light["h"])
        speed = np.linalg.norm(z[3:])
        if ok and speed < 1.075 and (best is None or speed > best[0]):
            best = speed, tip, z
    speed, tip, z = best
    say("speed", speed, "after the tip at", tip[0, 1:4] - q)
    assert speed > 1.04
    far = np.array([[0.5, *(z[:3] + 24.0 * z[3:] / speed), 0.1]])
    (ta, sa), (tb, sb) = run(np.concatenate([tip, far]))
    assert np.array_equal(ta["hit"], tb["hit"]) and np.abs(ta["hit"][0] - q).max() < 1e-6
    for k in sa:
        assert np.array_equal(sa[k], sb[k], equal_nan=True), (k, sa[k], sb[k])


@pytest.mark.parametrize("max_steps", [40, 300, 600, 900])
@pytest.mark.parametrize("w,h", [(24, 16), (160, 104)])
def test_shots_over_the_step_budget(rt, w, h, max_steps):
    """A pixel whose shot fails after some Newton steps (here: longer than
    max_steps) keeps the state of its last step, whichever launch it ends in: the
    same direction and length from two runs, and from the table padded to 33
    bumps, whose pixels end in another launch."""
    say("illumination", w, h, "max_steps", max_steps)
    wl = W.with_size(W.get("bumps16_1080p"), w, h)
    b = wl["metric"]["bumps"][0]
    pad = np.tile(np.array([[0.0, 3.0, 3.0, 3.0, 0.3]], np.float32), (33 - len(b), 1))
    res = [_run(rt, dict(wl, metric=dict(wl["metric"], bumps=m[None])), light=dict(LIGHT, max_steps=max_steps))[1]
           for m in (b, b, np.concatenate([b, pad]))]
    assert (res[0]["status"] == -1).any()
    for other in res[1:]:
        for k in other:
            assert np.array_equal(res[0][k], other[k], equal_nan=True), k


def test_packed_lists(rt):
    """The quadric's lists above the line where the iterations are packed again
    after each shot (16384 pixels): the geodesics found reach the light."""
    say("illumination, quadric 200x160, packed lists")
    wl = W.with_size(W.get("quadric_1080p"), 200, 160)
    tra, sh = _run(rt, wl)
    _check_found(wl, tra, sh, 0.9, sample=400)


def test_tiled_lists_equal_strips(rt):
    """Frames of more than 172032 pixels list them in 8x8 tiles, smaller ones in
    strips: three parameter sets of a frame with ragged sides, 177870 pixels in
    one call, against the sets one by one."""
    w, h = 245, 242
    say("illumination, 3 sets of %dx%d in tiles vs one by one" % (w, h))
    wl = W.with_size(W.get("adjoint_64x512", n_sets=3), w, h)
    _, sh = _run(rt, wl)
    n = w * h
    for s in range(3):
        one = dict(wl, metric=dict(wl["metric"], bumps=wl["metric"]["bumps"][s:s + 1]))
        _, shs = _run(rt, one)
        for k in ("status", "shade", "dir", "len"):
            assert np.array_equal(sh[k][s * n:(s + 1) * n], shs[k]), (s, k)
