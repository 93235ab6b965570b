"""The HIP path against the FP64 oracle at the sizes where a kernel's split
of the work changes: full and ragged blocks, the first and last size of a
rule's range.

Bars as in the other element-wise tests, from the same error budget: images
and A within 2e-5 of their maximum (hardware exp2 and FP32 rounding, ~1e-6
per term), gradients by cosine >= 0.9999 and relative L2 <= 1e-3 (a cell
within rounding of the footprint cutoff may add or drop its boundary term).
"""
import math

import numpy as np
import pytest
import torch

import oracle
from paper_2506_21633_amd import scenes

pytestmark = pytest.mark.gpu

ELEM = 2e-5
GRAD_COS = 0.9999
GRAD_L2 = 1e-3


def elem_err(a, ref):
    a, ref = np.asarray(a, np.float64), np.asarray(ref, np.float64)
    return float(np.abs(a - ref).max() / max(np.abs(ref).max(), 1e-300))


def spread_scene(seed, n, half, smin=0.05, smax=0.4):
    """n Gaussians over a box of the given half sides (seeded)."""
    rng = scenes.make_rng(seed)
    half = np.asarray(half, np.float64)
    return scenes.Scene(
        rng.uniform(-half, half, (n, 3)).astype(np.float32),
        np.exp(rng.uniform(math.log(smin), math.log(smax), (n, 3))).astype(np.float32),
        scenes.random_quats(rng, n), rng.uniform(0.2, 1.0, n).astype(np.float32),
        rng.uniform(1.0, 4.0, n).astype(np.float32))


def check(scene, views, cuda, options=None, grads=True, seed=0, **oracle_kw):
    from paper_2506_21633_amd import api
    g = api.GaussianTensors.from_numpy(scene, cuda)
    r = api.Renderer([g], views, options or api.RenderOptions())
    res = r.forward()
    A_ref, _, S_ref = oracle.forward(scene, views, **oracle_kw)
    A = r.intensity_shares(res).cpu().numpy().reshape(len(views), scene.n)
    for v in range(len(views)):
        if scene.n:
            assert elem_err(A[v], A_ref[v]) <= ELEM, v
        assert elem_err(res.image(v).cpu().numpy(), S_ref[v]) <= ELEM, v
    if not grads:
        r.status(res)
        return
    rng = np.random.default_rng(seed)
    G = [rng.standard_normal((v.img_h, v.img_w)) for v in views]
    flat = torch.as_tensor(np.concatenate([x.ravel() for x in G]).astype(np.float32), device=cuda)
    d = r.backward(res, flat)[0]
    r.status(res)
    ref, _ = oracle.backward(scene, views, G, **oracle_kw)
    for k, t in d.items():
        a, b = t.cpu().numpy().ravel().astype(np.float64), ref[k].ravel()
        if not np.any(b):
            assert not np.any(a), k
            continue
        assert float(a @ b / (np.linalg.norm(a) * np.linalg.norm(b))) >= GRAD_COS, k
        assert np.linalg.norm(a - b) / np.linalg.norm(b) <= GRAD_L2, k


def grid_view(tiles_x, tiles_y, spacing=0.2, incidence=45.0, azimuth=0.0):
    view = scenes.View.from_degrees(azimuth, incidence, 8, spacing)
    view.img_w, view.img_h = 8 * tiles_x, 8 * tiles_y
    return view


# Centres stay within 165 cells of the origin and Gaussians above 0.75 cells,
# where rounding a centre to FP32 moves a footprint by under 1e-5 of its peak.
@pytest.mark.parametrize("grids", [[(1, 1)], [(31, 33)], [(32, 32)], [(25, 41)],
                                   [(32, 32), (25, 41)]],
                         ids=lambda g: str(sum(a * b for a, b in g)))
def test_tile_worklist_blocks(cuda, grids):
    """Tile counts around the worklist's blocks of 1024 tiles."""
    views = [grid_view(a, b) for a, b in grids]
    wide = max(a for a, _ in grids), max(b for _, b in grids)
    scene = spread_scene(7, 1500, (0.5, 0.8 * wide[0], 0.5 * wide[1]), 0.15, 0.6)
    check(scene, views, cuda)


@pytest.mark.parametrize("kappa", [0.02, 3.0], ids=["thin", "opaque"])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 255, 256, 257, 1500])
def test_list_lengths(cuda, n, kappa):
    """One tile's list around the chunk (64) and the batch (4 chunks) of pass
    A, with few and with many hits per ray, stored for the backward, re-derived
    by it, and in the deterministic mode."""
    from paper_2506_21633_amd import api
    scene = spread_scene(n, n, (0.5, 0.7, 0.5), 0.15, 0.4)
    scene.ext[:] = np.float32(kappa) * scene.ext
    view = scenes.View.from_degrees(20.0, 40.0, 8, 0.2)
    for options in (api.RenderOptions(), api.RenderOptions(recompute=True),
                    api.RenderOptions(deterministic=True)):
        check(scene, [view], cuda, options)


@pytest.mark.parametrize("units", [0, 200, 16384, 5 * 16384])
def test_hit_stream_parts(cuda, units):
    """Streams of no, one, one full and five parts: tiles that find no room
    re-derive their hits, with the same gradients."""
    from paper_2506_21633_amd import api
    scene = spread_scene(11, 6000, (2.0, 9.0, 9.0), 0.15, 0.5)
    views = [grid_view(12, 12, 0.2, 45.0, a) for a in (0.0, 50.0)]
    g = api.GaussianTensors.from_numpy(scene, cuda)
    r = api.Renderer([g], views)
    cot = torch.as_tensor(np.random.default_rng(1).standard_normal(2 * 96 * 96)
                          .astype(np.float32), device=cuda)
    want = r.backward(r.forward(), cot)[0]
    plan = r.plan()
    plan.hit_bytes = min(plan.hit_bytes, 16 * units)
    res = r.forward(plan)
    got = r.backward(res, cot)[0]
    r.status(res)
    for k, t in want.items():   # FP32 rounding of re-derived against stored sums
        assert elem_err(got[k].cpu().numpy(), t.cpu().numpy()) <= 1e-5, k


@pytest.mark.parametrize("nq,nr", [(1, 1), (63, 129), (64, 257), (200, 40000), (4097, 511),
                                   (262080, 300), (262145, 129)])
@pytest.mark.parametrize("kind", ["box", "bad"])
def test_nearest_parts(cuda, nq, nr, kind):
    """Nearest neighbours where the references' split over parts begins and
    ends: the FP64 distances within FP32 rounding (1e-5 relative, and for the
    cancellation of coordinate differences 2^-22 of their size squared);
    points that are not finite are no one's neighbour and have none."""
    from scipy.spatial import cKDTree
    from paper_2506_21633_amd import train
    rng = np.random.default_rng(nq + 7 * nr)
    q = rng.uniform(-3, 3, (nq, 3)).astype(np.float32)
    ref = rng.uniform(-3, 3, (nr, 3)).astype(np.float32)
    if kind == "bad":
        ref[::5, 1], ref[1::7, 0], q[::9, 2], q[3::11, 0] = np.nan, np.inf, np.nan, -np.inf
    got = train.nearest_sq(torch.as_tensor(q, device=cuda),
                           torch.as_tensor(ref, device=cuda)).cpu().numpy()
    ok, qok = np.isfinite(ref).all(1), np.isfinite(q).all(1)
    assert np.isinf(got[~qok]).all()
    if not ok.any():
        assert np.isinf(got).all()
        return
    want = cKDTree(ref[ok].astype(np.float64)).query(q[qok].astype(np.float64))[0] ** 2
    assert (np.abs(got[qok] - want) <= 1e-5 * want + 2.0 ** -22 * 9.0).all()


@pytest.mark.parametrize("h,w", [(11, 11), (18, 42), (19, 43), (12, 75), (41, 200)])
@pytest.mark.parametrize("given", [True, False])
def test_image_metrics_tiles(cuda, h, w, given):
    """SSIM and PSNR where the tiles of 32 x 8 window positions end, the data
    range given or the references' maximum: within 1e-5 and 1e-4 of the
    reference (FP32 results of FP64 sums), the one-workgroup form of the
    call the same within FP32 rounding."""
    import ctypes
    from oracle import training as T
    from paper_2506_21633_amd import _capi as C
    from paper_2506_21633_amd import train
    rng = np.random.default_rng(h * w)
    ref = rng.gamma(2.0, 1.0, (3, h, w)).astype(np.float32)
    img = (ref + rng.normal(0, 0.4, ref.shape)).astype(np.float32)
    L = 5.0 if given else float(ref.max())
    x, y = torch.as_tensor(img, device=cuda), torch.as_tensor(ref, device=cuda)
    got = train.image_metrics(x, y, L if given else None)
    one = torch.full((3, 3), -1.0, device=cuda)
    C.check(C.lib().sdgr_image_metrics(
        x.data_ptr(), y.data_ptr(), 3, h, w, L, one[0].data_ptr(), one[1].data_ptr(),
        one[2].data_ptr(), ctypes.c_void_p(torch.cuda.current_stream(cuda).cuda_stream)))
    for k in range(3):
        assert abs(got["ssim_per"][k] - T.ssim(img[k], ref[k], L)) <= 1e-5, k
        assert abs(got["psnr_per"][k] - T.psnr(img[k], ref[k])) <= 1e-4, k
        assert abs(got["ssim_per"][k] - float(one[0, k])) <= 1e-6, k
    if not given:
        with pytest.raises(C.SDGRError):
            train.image_metrics(x, torch.zeros_like(y))


def run_views(scenes_, views, cuda, options, cots):
    """A, images and gradients per view set (one call)."""
    from paper_2506_21633_amd import api
    gs = [api.GaussianTensors.from_numpy(s, cuda) for s in scenes_]
    r = api.Renderer(gs, views, options)
    res = r.forward()
    A = r.intensity_shares(res).cpu().numpy()
    images = [res.image(v).cpu().numpy() for v in range(len(views))]
    flat = torch.as_tensor(np.concatenate([c.ravel() for c in cots]).astype(np.float32),
                           device=cuda)
    d = r.backward(res, flat)
    r.status(res)
    return A, images, [{k: t.cpu().numpy() for k, t in g.items()} for g in d]


@pytest.mark.parametrize("n", [1, 63, 64, 65, 8192, 8193, 16384, 16385])
def test_small_view_lists(cuda, n):
    """Views around the list-building kernels' record counts, beside a second
    scene of another count: the deterministic mode gives the same A, bit for
    bit, as in a call that also has a view too wide for these kernels (the
    sorts build every list then), and gradients and images within the
    rounding of FP32 sums; the other modes agree with it."""
    from paper_2506_21633_amd import api
    rng = np.random.default_rng(n)
    sc = [spread_scene(n, m, (2.0, 8.0, 8.0), 0.1, 0.3) for m in (n, max(n // 3, 1))]
    sc[0].means[:: 7] = sc[0].means[0]   # equal depths keep their order
    views = [grid_view(12, 12), grid_view(5, 30, azimuth=40.0), grid_view(9, 4, azimuth=80.0)]
    views[1].scene = 1
    wide = grid_view(257, 1, azimuth=10.0)
    cots = [rng.standard_normal((v.img_h, v.img_w)) for v in views]
    det = api.RenderOptions(deterministic=True)
    A, images, grads = run_views(sc, views, cuda, det, cots)
    A2, images2, grads2 = run_views(sc, views + [wide], cuda, det,
                                    cots + [np.zeros((wide.img_h, wide.img_w))])
    assert np.array_equal(A, A2[:A.size])
    for a, b in zip(images, images2):
        assert elem_err(a, b) <= 1e-6
    for g, g2 in zip(grads, grads2):
        for k in g:
            assert elem_err(g[k], g2[k]) <= 1e-5, k
    for options in (api.RenderOptions(), api.RenderOptions(recompute=True)):
        B, imagesB, gradsB = run_views(sc, views, cuda, options, cots)
        assert elem_err(B, A) <= ELEM
        for a, b in zip(imagesB, images):
            assert elem_err(a, b) <= ELEM
        for g, g2 in zip(gradsB, grads):
            for k in g:
                a, b = g[k].ravel().astype(np.float64), g2[k].ravel().astype(np.float64)
                assert np.linalg.norm(a - b) <= GRAD_L2 * np.linalg.norm(b), k


@pytest.mark.parametrize("n", [1, 64, 65, 513, 4000])
@pytest.mark.parametrize("deterministic", [False, True], ids=["any", "ordered"])
def test_images_without_lists(cuda, n, deterministic):
    """Small calls form their images without imaging-plane lists: against the
    oracle, ragged tiles and one view alone included; images that overlap in
    the buffer still add up (with atomics), and a plan with too few pairs is
    still refused."""
    from paper_2506_21633_amd import _capi as C
    from paper_2506_21633_amd import api
    scene = spread_scene(n + 3, n, (2.0, 6.0, 6.0), 0.1, 0.4)
    views = [grid_view(9, 7), grid_view(1, 13, azimuth=70.0), grid_view(6, 6, azimuth=33.0)]
    views[0].img_w, views[0].img_h = 69, 53   # ragged tiles
    g = api.GaussianTensors.from_numpy(scene, cuda)
    options = api.RenderOptions(deterministic=deterministic)
    r = api.Renderer([g], views, options)
    res = r.forward()
    r.status(res)
    _, _, want = oracle.forward(scene, views)
    for v in range(len(views)):
        alone = api.Renderer([g], views[v:v + 1], options).forward()
        assert elem_err(res.image(v).cpu().numpy(), want[v]) <= ELEM, v
        assert elem_err(alone.image(0).cpu().numpy(), want[v]) <= ELEM, v
    if not deterministic:
        both = api.Renderer([g], [views[2], grid_view(6, 6, azimuth=-20.0)], options)
        both.views_c[1].img_offset = 0
        _, _, add = oracle.forward(scene, [views[2], grid_view(6, 6, azimuth=-20.0)])
        assert elem_err(both.forward().images.reshape(-1)[:48 * 48].cpu().numpy(),
                        (add[0] + add[1]).ravel()) <= ELEM
    if n >= 513:
        plan = r.plan_for(r.plan().pairs_c, 100)
        with pytest.raises(C.SDGRError):
            r.status(r.forward(plan))


@pytest.mark.parametrize("nv", [9, 11, 12, 25])
def test_tables_over_launches(cuda, nv):
    """View tables that end in, at and after the first setup launch's data."""
    views = [grid_view(2, 1 + k % 3, azimuth=13.0 * k) for k in range(nv)]
    check(spread_scene(nv, 90, (1.0, 2.0, 2.0), 0.15, 0.5), views, cuda)


def test_emission_of_many_records(cuda):
    """Record counts below and at where the pair emission takes four blocks at
    a time, and one view further: in deterministic mode the common views' A
    agree bit for bit (their pairs have the same places), the images within
    the rounding of FP32 sums."""
    from paper_2506_21633_amd import api
    scene = spread_scene(5, 40000, (1.0, 3.0, 3.0), 0.03, 0.1)
    views = [grid_view(3 + k % 2, 4, azimuth=7.0 * k) for k in range(51)]
    g = api.GaussianTensors.from_numpy(scene, cuda)
    A, images = [], []
    for nv in (49, 50, 51):
        r = api.Renderer([g], views[:nv], api.RenderOptions(deterministic=True))
        res = r.forward()
        r.status(res)
        A.append(r.intensity_shares(res)[:49 * scene.n])
        images.append([res.image(v).cpu().numpy() for v in (0, 24, 48)])
    assert torch.equal(A[0], A[1]) and torch.equal(A[0], A[2])
    for got in images[1:]:
        for a, b in zip(got, images[0]):
            assert elem_err(a, b) <= 1e-6


def test_imaging_emission_of_many_records(cuda):
    """Record counts below and at where the imaging plane's emission takes 256
    records to a wave, the last block short, and views that end inside a
    block: the images of the views all three calls share agree in deterministic
    mode within the rounding of FP32 sums."""
    from paper_2506_21633_amd import api
    scene = spread_scene(8, 40003, (1.0, 3.0, 3.0), 0.03, 0.1)
    views = [grid_view(3 + k % 2, 4, azimuth=1.4 * k) for k in range(251)]
    g = api.GaussianTensors.from_numpy(scene, cuda)
    images = []
    for nv in (249, 250, 251):
        r = api.Renderer([g], views[:nv], api.RenderOptions(deterministic=True))
        res = r.forward()
        r.status(res)
        images.append(torch.cat([res.image(v).reshape(-1) for v in range(249)]))
    assert images[0].abs().max() > 0
    assert elem_err(images[1].cpu().numpy(), images[0].cpu().numpy()) <= 1e-6
    assert elem_err(images[2].cpu().numpy(), images[0].cpu().numpy()) <= 1e-6


@pytest.mark.parametrize("shadowing", [True, False], ids=["shadows", "none"])
@pytest.mark.parametrize("tiles", [(38, 40), (32, 48), (39, 41)], ids=lambda t: str(t[0] * t[1]))
def test_pass_a_by_number_of_tiles(cuda, tiles, shadowing):
    """Pass A around the number of tiles that changes its form (1536), with
    lists of a few entries to thousands, rays that stop early, and many hits
    of one ray in a batch."""
    from paper_2506_21633_amd import api
    a, b = tiles
    wide = (0.5, 0.8 * a, 0.8 * b / math.cos(math.radians(45.0)))
    scene = spread_scene(a, 15000, wide, 0.15, 0.6)
    scene.means[12000:] *= np.float32(0.03)                # a few crowded tiles
    scene.ext[13500:] *= np.float32(0.01)                  # that rays see far into
    check(scene, [grid_view(a, b)], cuda, api.RenderOptions(shadowing=shadowing),
          shadowing=shadowing)


@pytest.mark.parametrize("n", [16500, 262144, 262145, 1048576, 1048577])
def test_sort_tile_sizes(cuda, n):
    """Record counts around the change of the sorts' tiles: depth order and
    lists give the oracle's intensities."""
    scene = spread_scene(n, n, (1.0, 6.0, 6.0), 0.02, 0.05)
    check(scene, [grid_view(8, 8)], cuda, grads=False)


MODES = {"stored": {}, "recompute": {"recompute": True}, "ordered": {"deterministic": True}}


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("n,nv", [(16385, 1), (13000, 4)])
def test_one_tile_of_many_records(cuda, n, nv, mode):
    """Images of one tile each where the sorts build the lists: a view past
    the small views' record count, and views past their sum of pairs. The
    pair sort has one bucket and makes no pass."""
    from paper_2506_21633_amd import api
    scene = spread_scene(n, n, (0.5, 0.7, 0.5), 0.15, 0.4)
    views = [scenes.View.from_degrees(20.0 + 70.0 * k, 40.0, 8, 0.2) for k in range(nv)]
    check(scene, views, cuda, api.RenderOptions(**MODES[mode]))


@pytest.mark.parametrize("plane", ["computation", "imaging"])
@pytest.mark.parametrize("n", [262144, 262145])
def test_pairs_past_32_bits_overflow(cuda, n, plane):
    """Gaussians that have grown until each covers all 16384 tiles of a plane
    under a plan made for small ones: 2^32 pairs and 16384 more, which in 32
    bits would be none and few, are both reported."""
    from paper_2506_21633_amd import _capi as C
    from paper_2506_21633_amd import api
    scene = spread_scene(3, n, (1.0, 60.0, 60.0), 0.05, 0.1)
    scene.ext[:] = np.float32(1e-6)
    view = grid_view(128, 128)
    if plane == "imaging":   # one tile of rays, through every Gaussian
        view.comp_w = view.comp_h = 8
    g = api.GaussianTensors.from_numpy(scene, cuda)
    r = api.Renderer([g], [view], api.RenderOptions(shadowing=False))
    if plane == "computation":
        plan = r.plan()
    else:
        plan = r.plan_for(n, 20000)
    g.scales.fill_(300.0)
    res = r.forward(plan)
    with pytest.raises(C.SDGRError) as err:
        r.status(res)
    assert err.value.code == C.SDGR_EOVERFLOW
    if plane == "imaging":
        assert int((r.intensity_shares(res) > 0).sum()) == n   # all had pairs


@pytest.mark.parametrize("n", [1000, 4000, 20000])
def test_ordered_results_at_any_capacity(cuda, n):
    """Deterministic images and gradients do not depend on the pairs a plan
    has room for (the form of pass B is not chosen by them): an exact plan,
    one with headroom and one for far more pairs agree bit for bit."""
    from paper_2506_21633_amd import api
    scene = spread_scene(n + 5, n, (2.0, 6.0, 6.0), 0.1, 0.5)
    g = api.GaussianTensors.from_numpy(scene, cuda)
    views = [grid_view(9, 7), grid_view(6, 6, azimuth=33.0)]
    r = api.Renderer([g], views, api.RenderOptions(deterministic=True))
    exact = r.plan()
    cot = torch.as_tensor(np.random.default_rng(n).standard_normal(exact.image_floats)
                          .astype(np.float32), device=cuda)
    want = None
    for plan in (exact, r.planned(0.1), r.plan_for(exact.pairs_c, 3_000_000)):
        res = r.forward(plan)
        got = {"images": res.images, **r.backward(res, cot)[0]}
        r.status(res)
        want = want or got
        for k, t in got.items():
            assert torch.equal(t, want[k]), k


@pytest.mark.parametrize("opaque_views", [0, 7])
def test_hit_stream_reach(cuda, opaque_views):
    """A tile of many thin Gaussians stores its hits wherever the stream has
    room: the only tile of a call, and the one that starts in the last of
    eight parts, past seven longer lists that hardly use theirs. Its gradients
    are the oracle's."""
    from paper_2506_21633_amd import api
    thin = spread_scene(1, 20000, (0.5, 0.7, 0.5), 0.15, 0.4)
    thin.ext[:] *= np.float32(1e-4)
    dense = spread_scene(2, 40000, (0.5, 0.7, 0.5), 0.15, 0.4)
    dense.ext[:] *= np.float32(20.0)
    views = [scenes.View.from_degrees(40.0 * k, 40.0, 8, 0.2) for k in range(opaque_views + 1)]
    views[-1].scene = 1
    r = api.Renderer([api.GaussianTensors.from_numpy(s, cuda) for s in (dense, thin)], views)
    plan = r.plan()
    if opaque_views:
        plan.hit_bytes = 8 * 16384 * 16
    rng = np.random.default_rng(0)
    G = [rng.standard_normal((8, 8)) for _ in views]
    flat = torch.as_tensor(np.concatenate([x.ravel() for x in G]).astype(np.float32), device=cuda)
    api.count_work(True)
    try:
        res = r.forward(plan)
        d = r.backward(res, flat)[1]
        r.status(res)
        work = r.work_counters(res)
    finally:
        api.count_work(False)
    assert work["hits_a_fwd"] * 2 > 3 * 16384 * 16   # more than three parts hold
    assert work["tiles_a_bwd_rederived"] == 0
    assert work["tiles_a_bwd_stored"] == len(views)
    ref, _ = oracle.backward(thin, views[-1:], G[-1:])
    for k, t in d.items():
        a, b = t.cpu().numpy().ravel().astype(np.float64), ref[k].ravel()
        assert float(a @ b / (np.linalg.norm(a) * np.linalg.norm(b))) >= GRAD_COS, k
        assert np.linalg.norm(a - b) / np.linalg.norm(b) <= GRAD_L2, k


@pytest.mark.parametrize("units", [200, 16384, 3 * 16384])
def test_hit_stream_parts_of_many_tiles(cuda, units):
    """The same where a wave takes a tile (over 1536 tiles): streams that run
    out in some parts before others, with the bar of test_hit_stream_parts."""
    from paper_2506_21633_amd import api
    wide = (0.5, 0.8 * 40, 0.8 * 40 / math.cos(math.radians(45.0)))
    scene = spread_scene(13, 12000, wide, 0.15, 0.6)
    scene.means[9000:] *= np.float32(0.05)
    g = api.GaussianTensors.from_numpy(scene, cuda)
    r = api.Renderer([g], [grid_view(40, 40)])
    cot = torch.as_tensor(np.random.default_rng(1).standard_normal(320 * 320)
                          .astype(np.float32), device=cuda)
    want = r.backward(r.forward(), cot)[0]
    plan = r.plan()
    plan.hit_bytes = min(plan.hit_bytes, 16 * units)
    res = r.forward(plan)
    got = r.backward(res, cot)[0]
    r.status(res)
    for k, t in want.items():   # FP32 rounding of re-derived against stored sums
        assert elem_err(got[k].cpu().numpy(), t.cpu().numpy()) <= 1e-5, k


def test_infinite_cotangent(cuda):
    """An infinite cotangent of one pixel gives the amplitudes of the Gaussians
    that reach it an infinite gradient of its sign, as the sum that defines
    it, and leaves the others' as they are."""
    from paper_2506_21633_amd import api
    scene = spread_scene(4, 300, (1.0, 3.0, 3.0), 0.15, 0.5)
    view = grid_view(6, 5)
    rng = np.random.default_rng(4)
    g = api.GaussianTensors.from_numpy(scene, cuda)
    r = api.Renderer([g], [view])
    for sign in (1.0, -1.0):
        G = rng.standard_normal((view.img_h, view.img_w))
        G[19, 23] = sign * np.inf
        got = r.backward(r.forward(), torch.as_tensor(G.astype(np.float32), device=cuda))[0]
        a = got["amp"].cpu().numpy().astype(np.float64)
        want = oracle.backward(scene, [view], [G])[0]["amp"]
        far = np.isfinite(want)
        assert 0 < far.sum() < far.size
        assert np.array_equal(a[~far], want[~far])
        assert elem_err(a[far], want[far]) <= ELEM


@pytest.mark.parametrize("n", [300, 70000])
def test_images_with_a_gap_between_them(cuda, n):
    """Views moved apart in the image buffer, in a call without imaging-plane
    lists and one with them: the same images at their offsets, and zeros in
    the floats no view covers, whatever the buffer's memory held before."""
    from paper_2506_21633_amd import api
    scene = spread_scene(n, n, (1.0, 4.0, 4.0), 0.05, 0.2)
    g = api.GaussianTensors.from_numpy(scene, cuda)
    r = api.Renderer([g], [grid_view(5, 6), grid_view(4, 4, azimuth=30.0)])
    want = r.forward()
    gap, start = 101, 40 * 48
    r.views_c[1].img_offset = start + gap
    plan = r.plan()
    size = int(plan.image_floats)
    assert size == want.images.numel() + gap
    torch.full((size,), float("nan"), device=cuda)   # freed at once: the next one's memory
    images = r.forward(plan).images.cpu().numpy()
    assert np.all(images[start:start + gap] == 0.0)
    for v, off in ((0, 0), (1, start + gap)):
        img = want.image(v).cpu().numpy().ravel()
        assert elem_err(images[off:off + img.size], img) <= ELEM, v


@pytest.mark.parametrize("nv,n", [(49, 40003), (50, 40003), (260, 8009), (2, 1048583)])
def test_imaging_emission_rule(cuda, nv, n):
    """Records of few pairs below and past where the imaging plane's emission
    takes 256 to a wave, with view-major keys and (over 256 views) global
    ones: in deterministic mode the images are those of two calls with half
    the views each, within the rounding of FP32 sums."""
    from paper_2506_21633_amd import api
    scene = spread_scene(nv, n, (1.0, 3.0, 3.0), 0.005, 0.02)
    views = [grid_view(3 + k % 2, 4, azimuth=1.4 * k) for k in range(nv)]
    g = api.GaussianTensors.from_numpy(scene, cuda)
    options = api.RenderOptions(deterministic=True)

    def run(vs):
        r = api.Renderer([g], vs, options)
        plan = r.plan()
        assert plan.pairs_i < 1.69 * plan.records   # 2M records decide
        res = r.forward(plan)
        r.status(res)
        return res.images
    got, half = run(views), (nv + 1) // 2
    want = torch.cat([run(views[:half]), run(views[half:])])
    assert want.abs().max() > 0
    assert elem_err(got.cpu().numpy(), want.cpu().numpy()) <= 1e-6


# The small views' lists hold up to 16384 records a view and 256 tiles a side,
# and images form without lists up to 60000 records a view: these calls are
# past both, where the scans, the sorts and the emissions work.
MANY = 70000


@pytest.mark.parametrize("mode", ["stored", "ordered"])
@pytest.mark.parametrize("plane", ["computation", "imaging"])
def test_overflow_of_sorted_lists(cuda, plane, mode):
    """Too few pairs in the plan on one plane: reported by the scans, with a
    backward after it, and the exact plan renders as the oracle does."""
    from paper_2506_21633_amd import _capi as C
    from paper_2506_21633_amd import api
    scene = spread_scene(31, MANY, (1.0, 3.0, 3.0), 0.02, 0.1)
    views = [grid_view(6, 5), grid_view(4, 4, azimuth=100.0)]
    r = api.Renderer([api.GaussianTensors.from_numpy(scene, cuda)], views,
                     api.RenderOptions(**MODES[mode]))
    exact = r.plan()
    pairs = (exact.pairs_c // 2, exact.pairs_i) if plane == "computation" else (exact.pairs_c, 1000)
    res = r.forward(r.plan_for(*pairs))
    r.backward(res, torch.ones_like(res.images))
    with pytest.raises(C.SDGRError) as err:
        r.status(res)
    assert err.value.code == C.SDGR_EOVERFLOW
    ok = r.forward(exact)
    r.status(ok)
    _, _, want = oracle.forward(scene, views)
    for v in range(len(views)):
        assert elem_err(ok.image(v).cpu().numpy(), want[v]) <= ELEM, v


@pytest.mark.parametrize("mode", MODES)
def test_more_views_than_segments(cuda, mode):
    """Over 256 views with more tiles in all than the small views' lists take:
    one depth sort and one pair sort over all views, and imaging-plane keys
    that are global tile ids."""
    from paper_2506_21633_amd import api
    scene = spread_scene(18, 60, (0.6, 5.0, 4.0), 0.15, 0.4)
    views = [grid_view(12 + k % 2, 11, azimuth=1.4 * k) for k in range(260)]
    check(scene, views, cuda, api.RenderOptions(**MODES[mode]))


@pytest.mark.parametrize("mode", MODES)
def test_empty_views_between_sorted_ones(cuda, mode):
    """Views of an empty scene first, last and between views of others: empty
    segments of the sorts, blocks of records that end inside a view."""
    from paper_2506_21633_amd import api
    none = scenes.Scene(*(np.zeros((0,) + s, np.float32) for s in ((3,), (3,), (4,), (), ())))
    sc = [spread_scene(20, MANY, (1.0, 3.0, 3.0), 0.02, 0.1), none,
          spread_scene(21, 150, (1.0, 2.0, 2.0), 0.1, 0.3)]
    which = [1, 0, 1, 1, 2, 1, 0, 2, 1]
    views = [grid_view(4 + k % 2, 5, azimuth=25.0 * k) for k in range(len(which))]
    for v, s in zip(views, which):
        v.scene = s
    rng = np.random.default_rng(22)
    G = [rng.standard_normal((v.img_h, v.img_w)) for v in views]
    _, images, grads = run_views(sc, views, cuda, api.RenderOptions(**MODES[mode]), G)
    for s in (0, 2):
        mine = [k for k, x in enumerate(which) if x == s]
        vs = [scenes.View(**{**vars(views[k]), "scene": 0}) for k in mine]
        _, _, want = oracle.forward(sc[s], vs)
        for k, img in zip(mine, want):
            assert elem_err(images[k], img) <= ELEM, k
        ref, _ = oracle.backward(sc[s], vs, [G[k] for k in mine])
        for name, t in grads[s].items():
            a, b = t.ravel().astype(np.float64), ref[name].ravel()
            assert float(a @ b / (np.linalg.norm(a) * np.linalg.norm(b))) >= GRAD_COS, (s, name)
            assert np.linalg.norm(a - b) / np.linalg.norm(b) <= GRAD_L2, (s, name)
    for k, x in enumerate(which):
        if x == 1:
            assert not images[k].any(), k


def test_ordered_ragged_images_from_lists(cuda):
    """Ragged images of the deterministic mode through the workgroups that
    take a tile's list: edge tiles have lanes outside the image, which must
    still take part in the transpose of the masks. A view that only grazes
    Gaussian tails is held to the call's scale."""
    from paper_2506_21633_amd import api
    scene = scenes.vehicle(85, MANY)
    views = []
    for k, (w, h) in enumerate([(70, 52), (33, 17), (9, 61), (1, 5)]):
        v = scenes.View.from_degrees(40.0 + 70.0 * k, 35.0, w, 0.07)
        v.img_h = h
        views.append(v)
    r = api.Renderer([api.GaussianTensors.from_numpy(scene, cuda)], views,
                     api.RenderOptions(deterministic=True))
    res = r.forward()
    r.status(res)
    _, _, want = oracle.forward(scene, views)
    top = max(np.abs(S).max() for S in want)
    for v, S in enumerate(want):
        scale = max(np.abs(S).max(), 1e-3 * top)
        assert np.abs(res.image(v).cpu().numpy() - S).max() <= ELEM * scale, v


@pytest.mark.parametrize("nq,nr", [(1048576, 300), (1048641, 300), (2097088, 257), (2097153, 129)])
def test_nearest_of_many_queries(cuda, nq, nr):
    """Query counts where the references are last split in two parts and first
    not at all, and where the waves pass the number that is aimed at: the FP64
    distances, with the bar of test_nearest_parts."""
    from scipy.spatial import cKDTree
    from paper_2506_21633_amd import train
    rng = np.random.default_rng(nq + 7 * nr)
    q = rng.uniform(-3, 3, (nq, 3)).astype(np.float32)
    ref = rng.uniform(-3, 3, (nr, 3)).astype(np.float32)
    got = train.nearest_sq(torch.as_tensor(q, device=cuda),
                           torch.as_tensor(ref, device=cuda)).cpu().numpy()
    want = cKDTree(ref.astype(np.float64)).query(q.astype(np.float64), workers=8)[0] ** 2
    assert (np.abs(got - want) <= 1e-5 * want + 2.0 ** -22 * 9.0).all()
