"""The lag-domain spot kernel at every subaperture size it is compiled for (2 .. 12 pixels:
every transform length and lane grouping of its autocorrelation), against the FP64 oracle."""

import numpy as np
import pytest

import oracle
from wfs_cases import lgs_case, ngs_case, slope_tolerance

pytestmark = pytest.mark.gpu


def _forward(cfg, step, seed=42):
    import torch
    import paper_1608_00386_amd as W
    from wfs_cases import layers_for
    x = layers_for(cfg)
    out = {}
    for mode, flags in (("split", W.WFS_FLAG_SPLIT), ("footprint", W.WFS_FLAG_FOOTPRINT),
                        ("gather", W.WFS_FLAG_FUSED)):
        plan = W.Plan(cfg, flags=flags)
        s, a = plan.forward(torch.from_numpy(x).cuda(), step=step, seed=seed)
        out[mode] = (s.cpu().numpy().astype(np.float64), a.cpu().numpy().astype(np.float64))
    ref = oracle.forward(x.astype(np.float64), cfg, step, seed, noise=True)
    return out, ref


# (n_sub, N, bin): the smallest padding 2 n_sub, a wider one, images below and above 8 pixels
SIZES = [(2, 4, 1), (3, 6, 2), (3, 8, 1), (4, 8, 2), (5, 10, 1), (5, 12, 3), (6, 12, 2),
         (7, 14, 2), (7, 16, 4), (8, 16, 2), (8, 24, 3), (9, 18, 3), (9, 20, 2), (10, 20, 5),
         (10, 32, 4), (11, 22, 2), (11, 32, 4), (12, 24, 2), (12, 40, 4)]


@pytest.mark.parametrize("n_sub,N,b", SIZES)
@pytest.mark.parametrize("noise", [False, True])
@pytest.mark.parametrize("elong", [False, True])
def test_spots_of_every_subaperture_size_match_the_oracle(n_sub, N, b, noise, elong):
    if elong:
        cfg = lgs_case(5, n_sub, N, b, layers=2, n=96, pitch=0.25, noise=noise, n_sensors=2)
    else:
        cfg = ngs_case(5, n_sub, N, b, D=5.0 * n_sub * 0.1, obs=0.9, layers=2,
                       photons=900.0 if noise else 0.0, ro=2.0 if noise else 0.0, batch=2)
    got, (s_ref, a_ref) = _forward(cfg, 5)
    tol = slope_tolerance(cfg)
    for mode, (s, a) in got.items():
        worst = float((np.abs(s - s_ref) / tol[None, :]).max())
        assert worst <= 1.0, (mode, worst)
        np.testing.assert_allclose(a, a_ref, rtol=2e-5, atol=1e-4 * np.abs(a_ref).max(),
                                   err_msg=mode)
    assert np.array_equal(got["split"][0], got["footprint"][0])
    assert np.array_equal(got["split"][1], got["footprint"][1])


# images from 2 pixels (every lag in a class) to more pixels than the subaperture has (the
# axes through zero lag only), classes that leave and do not leave a remainder
ADJ = [(2, 4, 2), (3, 6, 1), (4, 8, 4), (5, 10, 2), (6, 12, 6), (7, 14, 7), (8, 16, 4),
       (8, 24, 2), (9, 18, 3), (10, 32, 4), (10, 20, 10), (11, 22, 2), (12, 24, 12), (12, 24, 3)]


@pytest.mark.parametrize("n_sub,N,b", ADJ)
@pytest.mark.parametrize("atomic", [False, True])
def test_adjoint_of_every_image_size_matches_the_oracle(n_sub, N, b, atomic):
    import torch
    import paper_1608_00386_amd as W
    from wfs_cases import layers_for
    cfg = lgs_case(5, n_sub, N, b, layers=2, n=96, pitch=0.25, n_sensors=2)
    x = layers_for(cfg)
    g = np.random.default_rng(3).standard_normal((1, 2 * sum(
        len(oracle.pupil_geometry(s)["valid"]) for s in cfg["sensors"]))).astype(np.float32)
    g[0, 1] = g[0, 1 + g.shape[1] // 4] = 0.0  # a subaperture without gradient
    plan = W.Plan(cfg, flags=W.WFS_FLAG_ADJOINT_ATOMIC if atomic else 0)
    xt, gt = torch.from_numpy(x).cuda(), torch.from_numpy(g).cuda()
    ref = oracle.adjoint(x.astype(np.float64), cfg, 3, g.astype(np.float64))
    s, a = plan.forward(xt, step=3)
    for fwd in ({}, dict(fwd_slopes=s, fwd_aux=a)):
        got = plan.adjoint(xt, gt, step=3, **fwd).cpu().numpy().astype(np.float64)
        assert np.linalg.norm(got - ref) <= 1e-4 * np.linalg.norm(ref)
        assert np.abs(got - ref).max() <= 1e-3 * np.abs(ref).max()
    zero = plan.adjoint(xt, torch.zeros_like(gt), step=3)  # nothing left from the calls before
    assert not zero.any()


# (n_sub, layers, image pixels): many layers, whose stencil taps take most of the LDS; images of
# one pixel (every lag in a class, no column classes) and of more pixels than the field's lags
@pytest.mark.parametrize("n_sub,layers,n_pix,atomic", [
    (10, 31, 8, False), (12, 20, 12, False), (10, 24, 14, False), (12, 18, 1, False),
    (12, 18, 1, True), (8, 2, 24, False), (8, 2, 24, True), (12, 4, 28, False)])
def test_adjoint_of_many_layers_and_large_images_matches_the_oracle(n_sub, layers, n_pix, atomic):
    import torch
    import paper_1608_00386_amd as W
    from wfs_cases import layers_for
    b = next(b for b in range(1, 99) if b * n_pix >= 2 * n_sub and b * n_pix % 2 == 0)
    cfg = lgs_case(5, n_sub, b * n_pix, b, layers=layers, n=96, pitch=0.25, n_sensors=2)
    x = layers_for(cfg)
    g = np.random.default_rng(3).standard_normal((1, oracle.n_slopes(cfg))).astype(np.float32)
    plan = W.Plan(cfg, flags=W.WFS_FLAG_ADJOINT_ATOMIC if atomic else 0)
    xt, gt = torch.from_numpy(x).cuda(), torch.from_numpy(g).cuda()
    ref = oracle.adjoint(x.astype(np.float64), cfg, 3, g.astype(np.float64))
    s, a = plan.forward(xt, step=3)
    for fwd in ({}, dict(fwd_slopes=s, fwd_aux=a)):
        got = plan.adjoint(xt, gt, step=3, **fwd).cpu().numpy().astype(np.float64)
        assert np.linalg.norm(got - ref) <= 1e-4 * np.linalg.norm(ref)
        assert np.abs(got - ref).max() <= 1e-3 * np.abs(ref).max()
