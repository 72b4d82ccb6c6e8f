"""GPU parity of the rasterizer (through the C ABI) against the FP64 oracle.

Bars: tile ids, per-tile lists and the depth order bit-exact; images max-abs 1e-4
(rgb, V, normal, T; depth in units of the scene half-extent) on pixels the oracle does
not flag as threshold-ambiguous; gradients per tensor max |g - g*| / max(|g*|,
1e-2 rms(g*)) <= 1e-3 with the upstream gradient zeroed on ambiguous pixels.
"""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle
import synth
import paper_2606_28581_amd as ss
from paper_2606_28581_amd import _lib
from gpu_common import (ATOMIC_ORDER_TOL, GRAD_KEYS, context, expand3, make_plan, oracle_settings, rel_err,
                        to_np)

pytestmark = pytest.mark.gpu


def scene_tiny(seed=7, views=((45, 38), (33, 29), (70, 17)), n=400, **kw):
    return synth.make_scene(synth.tiny(n_surfels=n, views=views, seed=seed, **kw))


# ---------------------------------------------------------------- binning
def check_binning(sc, ts):
    plan, surf, views = make_plan(sc, ts=ts)
    plan.forward(surf, views)
    b = plan.debug_binning(0)
    st = oracle_settings(ts=ts)
    order = oracle.depth_order(sc["surfels"]["mean"], sc["b_z"])
    np.testing.assert_array_equal(b["order"].astype(np.int64), order)
    toff, pairs = 0, []
    for v, (W, H) in enumerate(zip(sc["width"], sc["height"])):
        B, bb = oracle.view_camera(sc, v)
        _, _, _, tiles = oracle.binning(sc, B, bb, int(W), int(H), ts, st)
        np.testing.assert_array_equal(b["tiles"][v], tiles)
        ranges, flat = oracle.tile_lists(order, tiles, int(W), int(H), ts)
        nt = ranges.shape[0]
        gr = b["ranges"][toff:toff + nt].astype(np.int64)
        for t in range(nt):
            g = b["lists"][gr[t, 0]:gr[t, 1]].astype(np.int64)
            e = flat[ranges[t, 0]:ranges[t, 1]]
            np.testing.assert_array_equal(g, e, err_msg=f"view {v} tile {t}")
        empty = ranges[:, 1] == ranges[:, 0]
        assert np.all(gr[empty] == 0), f"view {v}: empty tiles carry (0, 0)"
        toff += nt
        pairs.append(len(flat))
    assert toff == b["ranges"].shape[0]
    return pairs


@pytest.mark.parametrize("ts", [8, 16, 32])
def test_binning_bit_exact(ts):
    check_binning(scene_tiny(seed=3, views=((71, 45), (40, 40), (17, 90)), n=700), ts)


def test_binning_bit_exact_with_a_view_that_sees_nothing():
    """A view whose camera is shifted far off the scene has no pairs: its run in the
    per-view tile sort is empty, and the views after it must still land in place."""
    sc = scene_tiny(seed=4, views=((52, 41), (40, 40), (33, 58)), n=600)
    sc["Fxy"] = sc["Fxy"].copy()
    sc["Fxy"][1, :, 3] += 1.0e5
    pairs = check_binning(sc, 8)
    assert pairs[1] == 0 and pairs[0] > 0 and pairs[2] > 0


def test_binning_bit_exact_many_sort_blocks_per_view():
    """Views whose pair runs span many 4096-pair sort blocks (and 2 radix passes)."""
    sc = scene_tiny(seed=9, views=((300, 221), (257, 311)), n=30000)
    pairs = check_binning(sc, 8)
    assert min(pairs) > 5 * 4096


def test_binning_bit_exact_with_32_bit_tile_keys():
    """Views of up to 2^16 tiles sort 16-bit tile keys local to the view; a 2080 x 2056
    view at 8 x 8 has 66,820 tiles, so this plan sorts 32-bit global keys."""
    sc = scene_tiny(seed=10, views=((2080, 2056), (60, 50)), n=3000, extent=40.0)
    pairs = check_binning(sc, 8)
    assert min(pairs) > 0


@pytest.mark.parametrize("n,nv", [(70_100, 30), (131_073, 13)])
def test_projection_of_several_views_a_block_equals_one_view_a_block(n, nv):
    """Many views of many surfels are projected four a block (the last group part-filled);
    a plan of some of the same views, one a block, must get the same records and tile ranges."""
    sc = scene_tiny(seed=17, n=n, views=tuple((9 + v % 3, 8 + v % 4) for v in range(nv)))
    plan, surf, views = make_plan(sc)
    plan.forward(surf, views)
    whole = plan.debug_binning(0, records=True)
    keys = ("width", "height", "Fxy", "dF", "colC", "colc", "ambient", "sun")
    for part in (slice(0, 2), slice(nv - 1, nv)):
        few = dict(sc, **{k: sc[k][part] for k in keys})
        plan, surf, views = make_plan(few)
        plan.forward(surf, views)
        b = plan.debug_binning(0, records=True)
        for k in ("tiles", "records"):
            np.testing.assert_array_equal(b[k], whole[k][part], k)


def test_records_centre_matches_fp64():
    sc = scene_tiny(seed=5)
    plan, surf, views = make_plan(sc)
    plan.forward(surf, views)
    rec = plan.debug_binning(0, records=True)["records"]
    st = oracle_settings()
    for v, (W, H) in enumerate(zip(sc["width"], sc["height"])):
        B, bb = oracle.view_camera(sc, v)
        c, _, _, _ = oracle.binning(sc, B, bb, int(W), int(H), 16, st)
        cg = rec[v][:, 2:4].astype(np.float64) + rec[v][:, 4:6].astype(np.float64)
        np.testing.assert_allclose(cg, c, rtol=1e-12, atol=1e-9)


# ---------------------------------------------------------------- forward
def check_forward(sc, out, ref, half_extent, tol=1e-4):
    W, H = sc["width"], sc["height"]
    ok = ~ref["ambiguous"]
    ok3 = expand3(ok, W, H)
    for k in ("image", "albedo", "normal"):
        err = np.abs(to_np(out[k])[ok3] - ref[k][ok3]).max()
        assert err <= tol, (k, err)
    for k in ("vis", "T"):
        err = np.abs(to_np(out[k])[ok] - ref[k][ok]).max()
        assert err <= tol, (k, err)
    err = np.abs(to_np(out["depth"])[ok] - ref["depth"][ok]).max() / half_extent
    assert err <= tol, ("depth", err)
    return ok.mean()


@pytest.mark.parametrize("ts,batch,mode", [(16, 64, 0), (8, 32, 0), (32, 256, 1), (16, 7, 0)])
def test_forward_multiview_ragged(ts, batch, mode):
    sc = scene_tiny(seed=11)
    plan, surf, views = make_plan(sc, ts=ts, batch=batch, mode=mode)
    out = plan.forward(surf, views)
    ref = oracle.forward(sc, oracle_settings(ts=ts, mode=mode))
    frac = check_forward(sc, out, ref, sc["spec"].extent / 2)
    assert frac > 0.99


def test_forward_with_visibility_channel():
    sc = scene_tiny(seed=12)
    vis = np.random.default_rng(1).uniform(size=(3, 400)).astype(np.float32)
    plan, surf, views = make_plan(sc)
    out = plan.forward(surf, views, torch.as_tensor(vis, device="cuda"))
    ref = oracle.forward(sc, oracle_settings(), vis=vis)
    check_forward(sc, out, ref, sc["spec"].extent / 2)


def test_forward_config1_full_image():
    """Plain-method tiny workload: 20k surfels, one 256x256 view, 16x16 tiles."""
    sc = synth.make_scene(synth.config(1))
    plan, surf, views = make_plan(sc)
    out = plan.forward(surf, views)
    ref = oracle.forward(sc, oracle_settings())
    frac = check_forward(sc, out, ref, sc["spec"].extent / 2)
    assert frac > 0.999
    assert (ref["T"] < 0.5).mean() > 0.5


# ---------------------------------------------------------------- backward
def check_backward(sc, plan, surf, views, out, ref, vis=None, tol=1e-3, mode=0):
    st = oracle_settings(mode=mode)
    dI, dD, dN = synth.upstream_grads(sc)
    W, H = sc["width"], sc["height"]
    amb = ref["ambiguous"]
    amb3 = expand3(amb, W, H)
    dI[amb3] = 0; dN[amb3] = 0; dD[amb] = 0
    t = lambda a: torch.as_tensor(a, device="cuda")
    g = plan.backward(surf, views, out, t(dI), t(dD), t(dN), vis=None if vis is None else t(vis))
    gref = oracle.backward(sc, dI, dD, dN, st, vis=vis)
    errs = {}
    for k in GRAD_KEYS:
        errs[k] = rel_err(to_np(g[k]), gref[k])
    bad = {k: e for k, e in errs.items() if e > tol}
    assert not bad, errs
    return errs


@pytest.mark.parametrize("ts,batch", [(16, 64), (8, 64), (8, 32), (8, 48), (8, 7), (32, 100)])
def test_backward_multiview_with_colour_and_vis(ts, batch):
    """8x8 tiles take the contributor-mask walk: batch 32 splits the forward's 64-position
    mask words, batch 48 and 7 make chunks that straddle two words."""
    sc = scene_tiny(seed=13)
    vis = np.random.default_rng(2).uniform(size=(3, 400)).astype(np.float32)
    plan, surf, views = make_plan(sc, ts=ts, batch=batch)
    out = plan.forward(surf, views, torch.as_tensor(vis, device="cuda"))
    ref = oracle.forward(sc, oracle_settings(ts=ts), vis=vis)
    check_backward(sc, plan, surf, views, out, ref, vis=vis)


def test_backward_8x8_without_contributor_masks():
    """A plan laid out for 16x16 tiles and switched to 8x8 has no room for contributor
    masks: the 8x8 backward then takes the box-test walk, which must give the same
    gradients."""
    sc = scene_tiny(seed=14)
    vis = np.random.default_rng(3).uniform(size=(3, 400)).astype(np.float32)
    plan, surf, views = make_plan(sc, ts=16, batch=64)
    # room for the 8x8 pairs in a workspace laid out at 16x16 (no mask words)
    plan.bind(8 * plan.cap_main, plan.cap_sun)
    plan.set_settings(ss.default_settings(tile_size=8, batch_depth=64))
    m, _ = plan.count_pairs(surf, views)
    assert m <= plan.cap_main
    out = plan.forward(surf, views, torch.as_tensor(vis, device="cuda"))
    ref = oracle.forward(sc, oracle_settings(ts=8), vis=vis)
    check_backward(sc, plan, surf, views, out, ref, vis=vis)


@pytest.mark.parametrize("ts,bound_at,n,mean_list", [
    (16, 16, 400, 0), (16, 16, 3000, 300),   # staged batches part-filled, and split across words
    (32, 32, 400, 0), (32, 32, 3000, 300),
    (16, 8, 3000, 300), (32, 8, 400, 0),     # no room for contributor masks: the box-test walk
])
def test_backward_of_larger_tiles_with_and_without_masks(ts, bound_at, n, mean_list):
    sc = scene_tiny(seed=15, n=n)
    vis = np.random.default_rng(5).uniform(size=(len(sc["width"]), n)).astype(np.float32)
    plan, surf, views = make_plan(sc, ts=bound_at)
    if ts != bound_at:
        plan.set_settings(ss.default_settings(tile_size=ts, batch_depth=64))
    m, _ = plan.count_pairs(surf, views)
    assert m <= plan.cap_main
    tiles = sum(-(-int(w) // ts) * -(-int(h) // ts) for w, h in zip(sc["width"], sc["height"]))
    assert m >= mean_list * tiles
    out = plan.forward(surf, views, torch.as_tensor(vis, device="cuda"))
    ref = oracle.forward(sc, oracle_settings(ts=ts), vis=vis)
    check_backward(sc, plan, surf, views, out, ref, vis=vis)


@pytest.mark.parametrize("ts", [8, 16])
def test_backward_of_a_small_and_of_a_large_launch(ts):
    """The same pixels as a view of their own (a wave per quadrant) and as the corner of a view
    of 17,161 blocks (a wave per block), with the upstream gradient on those pixels only."""
    S, L = 64, 1048
    small = scene_tiny(seed=19, views=((S, S),), n=800)
    up = synth.upstream_grads(small)
    grads = []
    for side in (S, L):
        sc = dict(small, width=np.array([side], np.int32), height=np.array([side], np.int32))
        d = []
        for x in up:
            full = np.zeros((x.size // (S * S), side, side), np.float32)
            full[:, :S, :S] = x.reshape(-1, S, S)
            d.append(torch.as_tensor(full.reshape(-1), device="cuda"))
        plan, surf, views = make_plan(sc, ts=ts)
        out = plan.forward(surf, views)
        grads.append(plan.backward(surf, views, out, *d))
    for k in GRAD_KEYS:
        assert rel_err(to_np(grads[1][k]), to_np(grads[0][k])) < 1e-3, k


@pytest.mark.parametrize("ts,dist,mode", [(32, False, 0), (32, False, 1), (16, False, 1), (8, False, 1),
                                          (8, True, 0), (16, True, 0), (32, True, 0)])
def test_backward_of_a_small_and_of_a_large_launch_of_every_variant(ts, dist, mode):
    """As above for 32x32 tiles, the distortion term and no low-pass floor."""
    S, L = 64, 1048
    small = scene_tiny(seed=19, views=((S, S),), n=800)
    up = (*synth.upstream_grads(small), np.random.default_rng(8).normal(size=S * S).astype(np.float32))
    grads = []
    for side in (S, L):
        sc = dict(small, width=np.array([side], np.int32), height=np.array([side], np.int32))
        d = []
        for x in up:
            full = np.zeros((x.size // (S * S), side, side), np.float32)
            full[:, :S, :S] = x.reshape(-1, S, S)
            d.append(torch.as_tensor(full.reshape(-1), device="cuda"))
        plan, surf, views = make_plan(sc, ts=ts, mode=mode)
        kw = dict(depth_scale=0.1) if dist else {}
        out = plan.forward(surf, views, **kw)
        grads.append(plan.backward(surf, views, out, *d[:3], **kw, **(dict(d_dist=d[3]) if dist else {})))
    for k in GRAD_KEYS:      # each within 1e-3 of the oracle by the bar of these tests
        assert rel_err(to_np(grads[1][k]), to_np(grads[0][k])) < 2e-3, k


def test_workspace_of_smaller_tiles_is_enough_for_larger_ones():
    """The bytes that 8x8 tiles need bind at 16x16 too (no room for contributor masks there)."""
    sc = scene_tiny(seed=18, n=2000)
    plan, surf, views = make_plan(sc, ts=8)
    caps, nbytes = (plan.cap_main, plan.cap_sun), plan.workspace.numel()
    plan.set_settings(ss.default_settings(tile_size=16, batch_depth=64))
    assert plan.workspace_size(*caps) > nbytes
    _lib.call("ss_plan_bind_workspace", plan.handle, C.c_void_p(plan.workspace.data_ptr()), nbytes, *caps)
    out = plan.forward(surf, views)
    check_backward(sc, plan, surf, views, out, oracle.forward(sc, oracle_settings(ts=16)))


def bind_smallest(plan):
    """Binds the plan's workspace again with the fewest bytes that are accepted."""
    caps = plan.cap_main, plan.cap_sun
    lo, hi = 0, plan.workspace_size(*caps)
    bind = lambda n: _lib.call("ss_plan_bind_workspace", plan.handle, C.c_void_p(plan.workspace.data_ptr()), n, *caps)
    while hi - lo > 1:
        mid = (lo + hi) // 2
        try:
            bind(mid)
            hi = mid
        except ss.SatSplatError:
            lo = mid
    bind(hi)
    return hi


@pytest.mark.parametrize("bound_at", [16, 32])
def test_8x8_tiles_on_a_workspace_bound_without_masks(bound_at):
    """The fewest bytes that 16x16 or 32x32 tiles accept have no room for contributor masks at
    8x8 either: forward, backward, a step and the autotuner run all the same after the switch."""
    sc = scene_tiny(seed=21)
    plan, surf, views = make_plan(sc, ts=bound_at)
    plan.bind(16 * plan.cap_main, 0)                  # room for the 8x8 pairs
    assert bind_smallest(plan) < plan.workspace_size(plan.cap_main, 0)
    plan.set_settings(ss.default_settings(tile_size=8, batch_depth=64))
    m, _ = plan.count_pairs(surf, views)
    assert m <= plan.cap_main
    out = plan.forward(surf, views)
    check_backward(sc, plan, surf, views, out, oracle.forward(sc, oracle_settings(ts=8)))
    up = [torch.as_tensor(x, device="cuda") for x in synth.upstream_grads(sc)]
    ref = {k: to_np(t) for k, t in plan.backward(surf, views, out, *up).items()}
    bufs = ss.StepBuffers(surf.mean.shape[0], views.width, views.height, with_sun=False, upstream=up)
    ss.step(plan, surf, views, bufs)
    for k in GRAD_KEYS:
        assert rel_err(to_np(bufs.grads[k]), ref[k]) < ATOMIC_ORDER_TOL, k
    table = (C.c_double * 36)()
    best, ms, sv, vv, io = _lib.RasterSettings(), C.c_double(), surf.c(), views.c(), bufs.c()
    _lib.call("ss_autotune", plan.handle, C.byref(sv), C.byref(vv), C.byref(io), 1, C.byref(best), C.byref(ms),
              C.cast(table, C.c_void_p), C.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert ms.value > 0 and sum(x > 0 for x in table[2::3]) == 10


@pytest.mark.parametrize("ts", [16, 32])
def test_workspace_without_masks_where_the_full_one_does_not_fit(ts, monkeypatch):
    """A card without room for the full size of 16x16 or 32x32 tiles still takes the plan."""
    sc = scene_tiny(seed=23, n=3000)
    plan, surf, views = make_plan(sc, ts=ts)
    cap, full = plan.cap_main, plan.workspace.numel()
    empty = torch.empty

    def small_card(*size, **kw):
        if kw.get("dtype") == torch.uint8 and size[0] >= full:
            raise torch.OutOfMemoryError("no room")
        return empty(*size, **kw)

    monkeypatch.setattr(torch, "empty", small_card)
    plan.bind(0, 0)
    plan.bind(cap, 0)
    assert plan.workspace.numel() < full
    out = plan.forward(surf, views)
    check_backward(sc, plan, surf, views, out, oracle.forward(sc, oracle_settings(ts=ts)))
    with pytest.raises(torch.OutOfMemoryError):
        plan.bind(64 * cap, 0)


@pytest.mark.parametrize("ts", [16, 32])
def test_capacity_after_a_change_of_tile_size_has_room_for_masks(ts):
    sc = scene_tiny(seed=22, n=3000)
    plan, surf, views = make_plan(sc, ts=8)
    plan.set_settings(ss.default_settings(tile_size=ts, batch_depth=64))
    plan.ensure_capacity(surf, views)
    full = plan.workspace_size(plan.cap_main, plan.cap_sun)
    assert plan.workspace.numel() >= full
    out = plan.forward(surf, views)
    check_backward(sc, plan, surf, views, out, oracle.forward(sc, oracle_settings(ts=ts)))
    # and back: smaller tiles need less, nothing is bound again
    ptr = plan.workspace.data_ptr()
    plan.set_settings(ss.default_settings(tile_size=8, batch_depth=64))
    plan.ensure_capacity(surf, views)
    assert plan.workspace.data_ptr() == ptr
    out = plan.forward(surf, views)
    check_backward(sc, plan, surf, views, out, oracle.forward(sc, oracle_settings(ts=8)))


@pytest.mark.parametrize("ts,n", [(16, 6000), (32, 6000), (32, 700)])
def test_blocks_of_a_tile_that_see_little_of_its_list(ts, n):
    """All surfels in a few pixels: most 8x8 blocks of a tile stage nothing from a list of more
    than 64 words, one stages nearly all of it.  Every pixel composites the same pairs in the
    same order at every tile size, so the forward's results are equal to the bit."""
    sc = scene_tiny(seed=16, views=((64, 64),), n=n)
    s = sc["surfels"]
    s["mean"][:, :2] = s["mean"][:, :2].mean(0) + 0.1 * (s["mean"][:, :2] - s["mean"][:, :2].mean(0))
    s["opacity"] *= 0.05
    t = lambda a: torch.as_tensor(a, device="cuda")
    up = [t(x) for x in synth.upstream_grads(sc)]
    res = {}
    for size in (8, ts):
        plan, surf, views = make_plan(sc, ts=size)
        out = plan.forward(surf, views)
        res[size] = out, plan.backward(surf, views, out, *up)
    b = plan.debug_binning(0)["ranges"].astype(np.int64)
    assert (b[:, 1] - b[:, 0]).max() > 0.7 * n
    for k in ("image", "albedo", "depth", "normal", "T"):
        assert torch.equal(res[ts][0][k], res[8][0][k]), k
    for k in GRAD_KEYS:      # each within 1e-3 of the oracle by the bar of these tests
        assert rel_err(to_np(res[ts][1][k]), to_np(res[8][1][k])) < 2e-3, k


def test_backward_config1():
    sc = synth.make_scene(synth.config(1))
    plan, surf, views = make_plan(sc)
    out = plan.forward(surf, views)
    ref = oracle.forward(sc, oracle_settings())
    check_backward(sc, plan, surf, views, out, ref)


def test_autograd_function_matches_plan_backward():
    """torch.autograd.Function around the library's adjoint: gradients of a loss through
    rasterize() equal the oracle's (upstream gradient zeroed on ambiguous pixels)."""
    import paper_2606_28581_amd as ss
    sc = scene_tiny(seed=14, views=((30, 30),), n=200)
    plan, surf, views = make_plan(sc)
    params = [surf.mean, surf.t_u, surf.t_v, surf.scale, surf.opacity, surf.albedo, views.dF,
              views.colC, views.colc, views.ambient]
    for p in params:
        p.requires_grad_(True)
    o = ss.rasterize(plan, views, surf)
    ref = oracle.forward(sc, oracle_settings())
    dI, dD, dN = synth.upstream_grads(sc)
    amb = ref["ambiguous"]
    amb3 = expand3(amb, sc["width"], sc["height"])
    dI[amb3] = 0; dN[amb3] = 0; dD[amb] = 0
    t = lambda a: torch.as_tensor(a, device="cuda")
    L = (o["image"] * t(dI)).sum() + (o["depth"] * t(dD)).sum() + (o["normal"] * t(dN)).sum()
    L.backward()
    gref = oracle.backward(sc, dI, dD, dN, oracle_settings())
    for k, p in zip(GRAD_KEYS, params):
        assert p.grad is not None, k
        assert rel_err(to_np(p.grad), gref[k]) < 1e-3, k


# ------------------------------------------------------- clamp and degenerate branches
@pytest.mark.parametrize("used", [("image",), ("depth",), ("normal",), ("depth", "normal")])
def test_autograd_of_some_outputs_is_the_adjoint_with_zeros_for_the_rest(used):
    sc = scene_tiny(seed=14, views=((30, 30), (17, 22)), n=300)
    plan, surf, views = make_plan(sc, ts=8)
    params = [surf.mean, surf.t_u, surf.t_v, surf.scale, surf.opacity, surf.albedo, views.dF,
              views.colC, views.colc, views.ambient]
    for p in params:
        p.requires_grad_(True)
    o = ss.rasterize(plan, views, surf)
    t = lambda a: torch.as_tensor(a, device="cuda")
    up = dict(zip(("image", "depth", "normal"), (t(x) for x in synth.upstream_grads(sc))))
    got = torch.autograd.grad([o[k] for k in used], params, [up[k] for k in used])
    ref = plan.backward(surf, views, {k: o[k] for k in ("albedo", "vis", "T", "last")},
                        *(x if k in used else torch.zeros_like(x) for k, x in up.items()))
    for k, g in zip(GRAD_KEYS, got):
        assert rel_err(to_np(g), to_np(ref[k])) < ATOMIC_ORDER_TOL, k


@pytest.mark.parametrize("ts,batch,mode", [(8, 64, 0), (8, 48, 1), (16, 64, 0), (16, 64, 1)])
def test_clamped_and_degenerate_surfels_forward_and_backward(ts, batch, mode):
    """Surfels with o G above alpha_max (alpha clamped to 0.99; the backward recovers T by
    dividing by 1 - 0.99) and degenerate surfels (edge-on in an oblique view, det T = 0
    exactly in a nadir view: no uv branch, low-pass disk only) at 8x8 (contributor-mask
    walk) and 16x16 (box walk) tiles, both low-pass modes."""
    from branch_scenes import branch_scene, special_surfels
    sc = branch_scene()
    n = sc["surfels"]["mean"].shape[0]
    V = len(sc["width"])
    vis = np.random.default_rng(3).uniform(size=(V, n)).astype(np.float32)
    plan, surf, views = make_plan(sc, ts=ts, batch=batch, mode=mode)
    out = plan.forward(surf, views, torch.as_tensor(vis, device="cuda"))
    st = oracle_settings(ts=ts, mode=mode)
    ref = oracle.forward(sc, st, vis=vis)
    check_forward(sc, out, ref, sc["spec"].extent / 2)
    # the clamp changes this scene's render (the branch is reached)
    noclamp = oracle.forward(sc, oracle.Settings(lowpass_mode=mode,
                                                 alpha_max=np.float32(0.99999).item()), vis=vis)
    assert np.abs(noclamp["image"] - ref["image"]).max() > 1e-3
    errs = check_backward(sc, plan, surf, views, out, ref, vis=vis, mode=mode)
    clamp, deg = special_surfels(sc)
    gref = oracle.backward(sc, *synth.upstream_grads(sc), st, vis=vis)
    assert np.abs(gref["mean"][deg]).max() > 0 and np.abs(gref["albedo"][clamp]).max() > 0


def test_graph_is_invalidated_by_rebinding_and_settings_changes():
    """A captured graph holds raw workspace pointers: after the plan's workspace is
    rebound, or its settings change, a replay is refused instead of running stale."""
    import paper_2606_28581_amd as ss
    sc = scene_tiny(seed=15)
    plan, surf, views = make_plan(sc)
    dI, dD, dN = [torch.as_tensor(x, device="cuda") for x in synth.upstream_grads(sc)]
    bufs = ss.StepBuffers(surf.mean.shape[0], views.width, views.height, with_sun=False,
                          upstream=(dI, dD, dN))
    g = ss.Graph(plan, surf, views, bufs)
    g.launch(check=True)
    torch.cuda.synchronize()
    plan.bind(plan.cap_main + 4096, plan.cap_sun)
    with pytest.raises(ss.SatSplatError):
        g.launch()
    g2 = ss.Graph(plan, surf, views, bufs)
    g2.launch(check=True)
    plan.set_settings(ss.default_settings(tile_size=8, batch_depth=32))
    with pytest.raises(ss.SatSplatError):
        g2.launch()
    torch.cuda.synchronize()


# ---------------------------------------------------------------- edge cases
def test_empty_scene_gives_background():
    sc = scene_tiny(seed=1, views=((20, 13),), n=10)
    sc["surfels"] = {k: v[:0] for k, v in sc["surfels"].items()}
    plan, surf, views = make_plan(sc)
    out = plan.forward(surf, views)
    assert np.all(to_np(out["T"]) == 1.0) and np.all(to_np(out["albedo"]) == 0.0)
    ref = oracle.forward(sc, oracle_settings())
    np.testing.assert_allclose(to_np(out["image"]), ref["image"], atol=1e-6)
    g = plan.backward(surf, views, out, *[torch.ones(k, device="cuda") for k in (3 * 260, 260, 3 * 260)])
    assert np.all(np.isfinite(to_np(g["colC"])))


def test_transparent_surfels_and_single_pixel_views():
    sc = scene_tiny(seed=2, views=((1, 1), (1, 9), (16, 16), (17, 1)), n=300)
    sc["surfels"]["opacity"][:100] = np.float32(0.5 / 255)
    plan, surf, views = make_plan(sc)
    out = plan.forward(surf, views)
    ref = oracle.forward(sc, oracle_settings())
    check_forward(sc, out, ref, sc["spec"].extent / 2)
    b = plan.debug_binning(0)
    assert np.all(b["tiles"][:, :100, 0] > b["tiles"][:, :100, 1])


def test_capacity_overflow_regrows_and_matches():
    sc = scene_tiny(seed=4)
    plan, surf, views = make_plan(sc)
    ref_out = {k: v.clone() for k, v in plan.forward(surf, views).items()}
    plan.bind(1, 0)                 # capacity of one pair
    out = plan.forward(surf, views, check=True)
    assert plan.regrows >= 1
    for k in ("image", "depth", "normal", "T"):
        np.testing.assert_array_equal(to_np(out[k]), to_np(ref_out[k]))


@pytest.mark.parametrize("ts", [8, 16])
def test_forward_deterministic_backward_nearly(ts):
    """The forward is bitwise reproducible; the backward's float atomics reorder sums, so
    repeated backwards differ by rounding only.  Prints the measured spread over 8 runs."""
    sc = scene_tiny(seed=6)
    plan, surf, views = make_plan(sc, ts=ts)
    a = {k: to_np(v) for k, v in plan.forward(surf, views).items()}
    out = plan.forward(surf, views)
    for k in a:
        np.testing.assert_array_equal(to_np(out[k]), a[k])
    dI, dD, dN = [torch.as_tensor(x, device="cuda") for x in synth.upstream_grads(sc)]
    g1 = {k: to_np(v).copy() for k, v in plan.backward(surf, views, out, dI, dD, dN).items()}
    spread = {k: 0.0 for k in GRAD_KEYS}
    for _ in range(8):
        g2 = plan.backward(surf, views, out, dI, dD, dN)
        for k in GRAD_KEYS:
            spread[k] = max(spread[k], rel_err(to_np(g2[k]), g1[k]))
    print(f"atomic-order spread ts={ts}: " + ", ".join(f"{k} {v:.2e}" for k, v in spread.items()))
    for k in GRAD_KEYS:
        assert spread[k] < ATOMIC_ORDER_TOL, k


def test_pair_count_scan_beyond_one_pass_of_the_partials_kernel():
    """More than 1024 x 4096 (view, surfel) slots: the pair-count scan's chunk totals
    take several passes of its single-block kernel (regression: the per-wave LDS array
    was sized for 4 of its 16 waves, so the carry broke after the first pass)."""
    views = tuple((24 + (v % 5), 20 + (v % 7)) for v in range(40))
    sc = synth.make_scene(synth.tiny(n_surfels=110_000, views=views, seed=41, colour=False,
                                     suns=False))
    assert 110_000 * 40 > 1024 * 4096
    plan, surf, views_t = make_plan(sc)
    K, _ = plan.count_pairs(surf, views_t)
    st = oracle_settings()
    expect = 0
    per_view = []
    for v, (W, H) in enumerate(zip(sc["width"], sc["height"])):
        B, bb = oracle.view_camera(sc, v)
        _, _, _, tiles = oracle.binning(sc, B, bb, int(W), int(H), 16, st)
        cnt = np.where(tiles[:, 0] <= tiles[:, 1],
                       (tiles[:, 1] - tiles[:, 0] + 1) * (tiles[:, 3] - tiles[:, 2] + 1), 0)
        per_view.append(tiles)
        expect += int(cnt.sum())
    assert K == expect
    plan.forward(surf, views_t)
    b = plan.debug_binning(0)
    for v in (0, 17, 39):
        np.testing.assert_array_equal(b["tiles"][v], per_view[v])
    assert b["lists"].shape[0] == expect


@pytest.mark.parametrize("ts", [8, 16])
def test_heavy_first_tile_order_changes_no_pixel(ts):
    """The heavy-tiles-first dispatch order against the static XCD order (default): every
    forward output and sun-depth texel bit-identical, gradients equal up to the atomics'
    summation order (the parity bar).  Two views of 600 x 520 px give more than one 4096-tile round of
    XCD chunks at 8 x 8."""
    sc = synth.make_scene(synth.tiny(n_surfels=4000, views=((600, 520), (520, 600)), extent=60.0,
                                     n_boxes=6, seed=15))
    res = {}
    for order in (0, 1):
        surf, views = ss.scene_to_device(sc, with_sun=True)
        st = ss.default_settings(tile_size=ts, batch_depth=64, sun_map_size=256, tile_order=order)
        plan = ss.Plan(context(), surf.mean.shape[0], views.width, views.height, st)
        plan.ensure_capacity(surf, views)
        D = torch.empty(2, 256, 256, device="cuda")
        vis = plan.shadow(surf, views, sun_depth=D)
        out = plan.forward(surf, views, vis)
        dI, dD, dN = [torch.as_tensor(x, device="cuda") for x in synth.upstream_grads(sc)]
        g = plan.backward(surf, views, out, dI, dD, dN, vis=vis)
        res[order] = ({k: to_np(v) for k, v in out.items()}, to_np(D), to_np(vis),
                      {k: to_np(v) for k, v in g.items()})
    (o0, D0, v0, g0), (o1, D1, v1, g1) = res[0], res[1]
    for k in o0:
        np.testing.assert_array_equal(o1[k], o0[k], err_msg=k)
    np.testing.assert_array_equal(D1, D0)
    np.testing.assert_array_equal(v1, v0)
    # the gradients' float atomics sum in a different order: held to the parity bar
    # (rel 1e-3); measured 1.1e-4 on t_u at tile 8
    for k in GRAD_KEYS:
        err = rel_err(g1[k], g0[k])
        print(f"tile order 0 vs 1, ts {ts}: {k} {err:.2e}")
        assert err < 1e-3, k


@pytest.mark.parametrize("n,views,slack", [
    (1, 1, 0),                 # one item
    (1023, 2, 0), (1025, 2, 0),            # around one block of 1024 items
    (130_049, 1, 0), (131_073, 3, 0),      # last size of 1024-item blocks, first of 2048
    (523_000, 1, 0), (523_500, 1, 0),      # 2048 -> 4096 items a block
    (1_045_000, 1, 0), (1_050_000, 1, 0),  # few blocks -> the three-kernel scans
    (40_000, 70, 0),                       # more views than some segments have blocks
    (9_000, 2, 3_000_000)])                # a capacity far beyond the pairs: empty blocks
def test_depth_order_and_tile_lists_across_sort_sizes(n, views, slack):
    """Order, tile lists and ranges against a stable numpy sort (integers: exact).  Quantised
    altitudes give long runs of equal depth keys, which must stay in index order."""
    rng = np.random.default_rng(n + views)
    f = lambda a: torch.as_tensor(np.ascontiguousarray(a, np.float32), device="cuda")
    mean = np.stack([rng.uniform(-30, 30, n), rng.uniform(-30, 30, n), np.round(rng.normal(size=n) * 8) / 4], 1)
    mean[:, 2] = np.where(rng.uniform(size=n) < 0.5, mean[:, 2], rng.normal(size=n))
    eye = np.tile(np.eye(3)[None], (n, 1, 1))
    surf = ss.SurfelTensors(f(mean), f(eye[:, 0]), f(eye[:, 1]), f(rng.uniform(0.02, 0.3, (n, 2))),
                            f(rng.uniform(0.01, 0.9, n)), f(rng.uniform(size=(n, 3))))
    W = np.full(views, 61, np.int32)
    H = np.full(views, 47, np.int32)
    F = np.zeros((views, 2, 4), np.float32)
    F[:, 0, 0], F[:, 1, 1] = 1.0, 0.8
    F[:, 0, 3], F[:, 1, 3] = 30.5 + np.arange(views) * 0.25, 23.5
    F[views // 2, 0, 3] = 1e6 if views > 2 else F[views // 2, 0, 3]        # one view sees nothing
    vt = ss.ViewTensors(W, H, f(F), 12.0)
    plan = ss.Plan(context(), n, W, H, ss.default_settings(tile_size=8, batch_depth=64))
    plan.ensure_capacity(surf, vt)
    if slack:
        plan.bind(plan.cap_main + slack, 0)
    plan.forward(surf, vt)
    b = plan.debug_binning(0)
    key = np.float32(12.0) - mean.astype(np.float32)[:, 2]
    order = np.argsort(key, kind="stable")
    np.testing.assert_array_equal(b["order"], order)
    tx = 8
    keys, who, off = [], [], 0
    for v in range(views):
        t = b["tiles"][v][order]
        nx, ny = np.maximum(t[:, 1] - t[:, 0] + 1, 0), np.maximum(t[:, 3] - t[:, 2] + 1, 0)
        for dy in range(int(ny.max(initial=0))):
            for dx in range(int(nx.max(initial=0))):
                m = np.nonzero((dx < nx) & (dy < ny))[0]
                keys.append(off + (t[m, 2] + dy).astype(np.int64) * tx + t[m, 0] + dx)
                who.append(m)
        off += tx * 6
    keys, who = np.concatenate(keys), np.concatenate(who)
    o = np.lexsort((who, keys))
    assert b["lists"].shape[0] == keys.size
    np.testing.assert_array_equal(b["lists"], order[who[o]])
    cnt = np.bincount(keys, minlength=off)
    end = np.cumsum(cnt)
    expect = np.where(cnt[:, None] > 0, np.stack([end - cnt, end], 1), 0)
    np.testing.assert_array_equal(b["ranges"], expect)


@pytest.mark.parametrize("n", [63, 1024, 2047, 2049, 32_767, 32_768, 32_769])
def test_depth_order_around_the_sizes_of_merged_chunks(n):
    """Whole chunks of 1024, one item less and more, and the last size that is merged."""
    test_depth_order_and_tile_lists_across_sort_sizes(n, 1, 0)


def test_backward_writes_gradients_directly_and_by_rows():
    """Up to 65,536 surfels the projection backward writes the gradient arrays itself, beyond
    by way of rank-ordered rows: one transparent surfel more must change nothing."""
    sc = synth.make_scene(synth.tiny(n_surfels=65_536, views=((131, 120), (90, 77)), extent=120.0, seed=12))
    more = dict(sc, surfels={k: np.concatenate([a, a[-1:]]) for k, a in sc["surfels"].items()})
    more["surfels"]["opacity"] = more["surfels"]["opacity"].copy()
    more["surfels"]["opacity"][-1] = 0.0
    dI, dD, dN = (torch.as_tensor(a, device="cuda") for a in synth.upstream_grads(sc))
    out = []
    for scene in (sc, more):
        plan, surf, views = make_plan(scene, ts=8)
        fwd = plan.forward(surf, views)
        g = plan.backward(surf, views, fwd, dI, dD, dN)
        out.append({k: to_np(t).copy() for k, t in g.items()})
    for k in GRAD_KEYS:
        a, b = out[0][k], out[1][k]
        if k in ("mean", "t_u", "t_v", "scale", "opacity", "albedo"):
            assert not b[-1].any()
            b = b[:-1]
        assert rel_err(b, a) <= ATOMIC_ORDER_TOL, k


@pytest.mark.parametrize("ts", [8, 16, 32])
def test_surfel_too_small_for_fp32_without_the_low_pass_floor(ts):
    """A frame whose inverse leaves FP32 (Q infinite), centred on a pixel's centre, so that Q
    delta is NaN there.  Without the low-pass floor such a pair has no weight, and no output may
    see it: the render equals the one in which the surfel is transparent."""
    f = lambda a: torch.as_tensor(np.ascontiguousarray(a, np.float32), device="cuda")
    F = np.zeros((1, 2, 4), np.float32)
    F[0, 0, 0] = F[0, 1, 1] = 0.125                  # exact: both centres are at (4.5, 4.5) px
    eye = np.tile(np.eye(3)[None], (2, 1, 1))
    v = ss.ViewTensors(np.array([24], np.int32), np.array([17], np.int32), f(F), 10.0)
    res = []
    for o in (0.9, 0.0):
        surf = ss.SurfelTensors(f([[36, 36, 3], [36, 36, 0]]), f(eye[:, 0]), f(eye[:, 1]),
                                f([[2e-38, 2e-38], [16, 16]]), f([o, 0.8]), f([[1, 0, 0], [0, 1, 0]]))
        plan = ss.Plan(context(), 2, v.width, v.height,
                       ss.default_settings(tile_size=ts, batch_depth=64, lowpass_mode=1))
        plan.ensure_capacity(surf, v)
        res.append({**plan.forward(surf, v, depth_scale=0.1), **{k + "_plain": t for k, t in plan.forward(surf, v).items()}})
        if o:
            rec = plan.debug_binning(0, records=True)["records"][0, 0]
            assert np.isinf(rec[8]) and np.isinf(rec[11]) and np.array_equal(rec[2:6], [4.5, 4.5, 0, 0])
    for k in res[0]:
        if not k.startswith("last"):                 # positions count the opaque one's list entry
            same = torch.equal(res[0][k], res[1][k]) and bool(torch.isfinite(res[0][k]).all())
            assert same, k
