"""The FFT-path spot kernels at the edges of their sizes (1, 2 and 4 spectrum chunks per axis;
fields that fill, half fill and just enter a 32-pixel block), several chunk counts in one
plan, against the FP64 oracle."""

import numpy as np
import pytest

import oracle
import synth
from wfs_cases import layers_for, ngs_case, slope_tolerance

pytestmark = pytest.mark.gpu


def _check(cfg, flags=0, step=2):
    import torch
    import paper_1608_00386_amd as W
    x = layers_for(cfg)
    plan = W.Plan(cfg, flags=flags)
    assert all(q == 1 for q in plan.paths)
    s, a = plan.forward(torch.from_numpy(x).cuda(), step=step, seed=9)
    s_ref, a_ref = oracle.forward(x.astype(np.float64), cfg, step, 9, noise=True)
    err = np.abs(s.cpu().numpy().astype(np.float64) - s_ref) / slope_tolerance(cfg)[None, :]
    assert err.max() <= 1.0, err.max()
    np.testing.assert_allclose(a.cpu().numpy(), a_ref, rtol=2e-5, atol=1e-4 * np.abs(a_ref).max())


@pytest.mark.parametrize("n_sub,N,b", [(13, 32, 1), (16, 32, 2), (16, 32, 8), (17, 64, 2),
                                       (31, 64, 2), (32, 64, 2), (24, 128, 4), (32, 128, 4),
                                       (33, 128, 4), (63, 128, 4), (64, 128, 4)])
@pytest.mark.parametrize("noise", [False, True])
def test_fft_path_sizes_match_the_oracle(n_sub, N, b, noise):
    _check(ngs_case(3, n_sub, N, b, D=9.0, obs=2.0, layers=2, n=96, pitch=0.2,
                    photons=3000.0 if noise else 0.0, ro=2.0 if noise else 0.0, batch=2))


@pytest.mark.parametrize("n_sub,N,b", [(2, 16, 1), (5, 16, 4), (8, 16, 2), (12, 32, 4)])
def test_small_fields_on_the_fft_path_match_the_oracle(n_sub, N, b):
    import paper_1608_00386_amd as W
    _check(ngs_case(9, n_sub, N, b, D=9.0, obs=2.0, layers=1, n=96, pitch=0.2, photons=500.0,
                    ro=2.0), flags=W.WFS_FLAG_FORCE_FFT)


def test_sensors_of_every_chunk_count_in_one_plan_match_the_oracle():
    cfg = ngs_case(2, 64, 128, 4, D=9.0, obs=2.0, layers=2, n=96, pitch=0.2, photons=4000.0,
                   ro=3.0, batch=3)
    for n_sa, n_sub, N, b in ((5, 14, 32, 4), (3, 20, 64, 2), (2, 40, 128, 4)):
        s = dict(cfg["sensors"][0])
        s.update(n_sa=n_sa, n_sub=n_sub, n_fft=N, bin=b, theta_x_rad=1e-5 * n_sub,
                 theta_y_rad=-2e-5, tilt_x_rad=3e-8, tilt_y_rad=-1e-8)
        cfg["sensors"].append(s)
    _check(cfg)
