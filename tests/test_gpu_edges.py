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


@pytest.mark.parametrize("tiles", [1, 1023, 1024, 1025, 2049])
def test_tile_worklist_blocks(cuda, tiles):
    """Strips of tiles around the worklist's blocks of 1024 tiles."""
    view = scenes.View.from_degrees(0.0, 45.0, 8, 0.2)
    view.img_w = 8 * tiles
    scene = spread_scene(tiles, 1500, (0.5, 0.8 * tiles, 0.5))
    check(scene, [view], cuda)
