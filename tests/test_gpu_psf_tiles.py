"""The PSF passes over several pupil columns a workgroup against one column a workgroup."""

import numpy as np
import pytest

import oracle
import synth
from synth.configs import ARCSEC

pytestmark = pytest.mark.gpu


def _system(ragged):
    """Two fine layers (one of odd size, wrapping under the pupil), a coarse zero-boundary one."""
    layers = [dict(nx=64, ny=64, pitch_m=0.25, alt_m=0.0, vx_mps=5.0, vy_mps=-3.0, weight=1.0,
                   boundary=0),
              dict(nx=49 if ragged else 48, ny=47, pitch_m=0.3, alt_m=6000.0, vx_mps=-8.0,
                   vy_mps=2.0, weight=1.0, boundary=0),
              dict(nx=9, ny=9, pitch_m=1.0, alt_m=2000.0, vx_mps=0.0, vy_mps=0.0, weight=-1.0,
                   boundary=1)]
    offs, stride = synth.layer_offsets(layers, 64)
    for layer, o in zip(layers, offs):
        layer["offset"] = o
    cfg = dict(layers=layers, layer_stride=stride, lambda_ref_m=0.5e-6, dt_s=0.002)
    rng = np.random.default_rng(11)
    return cfg, (rng.standard_normal(stride) * 0.8).astype(np.float32)


# pupils of at most half of the transform and of more, sizes around the phase's 64 x 32 tiles
# and no multiples of the passes' columns; enough stars for several columns a workgroup
@pytest.mark.parametrize("n_pup,N,ragged", [(8, 16, False), (13, 16, True), (16, 32, False),
                                            (31, 32, True), (33, 64, True), (64, 256, False),
                                            (65, 128, True), (97, 512, False), (300, 512, True),
                                            (130, 1024, True), (129, 2048, False)])
def test_star_does_not_depend_on_the_others(n_pup, N, ragged):
    """An image of a plan of many stars has the bits of the plan of that star alone (which the
    oracle checks), and its variance too."""
    import torch
    import paper_1608_00386_amd as W
    cfg, x = _system(ragged)
    D, obs, lam = 0.25 * n_pup, 0.06 * n_pup, [1.2e-6]
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    S = min(256, 2 * cus * 4 // n_pup + 5)
    stars = [(0.3 * k * ARCSEC, -0.2 * k * ARCSEC) for k in range(S)]
    xt = torch.from_numpy(x).cuda()
    many = W.PsfPlan(cfg, stars, D, obs, n_pup, lam, [N])
    psf, var = many.buffers()
    for step in (3, 40):
        many.accumulate(xt, step, psf, var)
    for k in (0, 1, S - 1):
        one = W.PsfPlan(cfg, [stars[k]], D, obs, n_pup, lam, [N])
        p1, v1 = one.buffers()
        for step in (3, 40):
            one.accumulate(xt, step, p1, v1)
        assert torch.equal(many.image(psf, 0, k), one.image(p1, 0, 0)), k
        v = float(v1.reshape(-1)[0])  # (its double sums are grouped by the size of the plan)
        assert abs(float(var.reshape(-1)[k]) - v) <= 1e-11 * v, k
    want, ref_var = oracle.long_exposure(x.astype(np.float64), cfg, [stars[S - 1]], [3, 40], lam,
                                         [N], D, obs, n_pup)
    pdl = many.n_lit / N ** 2
    got = many.image(psf, 0, S - 1).cpu().numpy().astype(np.float64)
    assert np.abs(got - want[0, 0]).max() <= 2e-5 * 2 * pdl
    assert abs(float(var.reshape(-1)[S - 1]) - ref_var[0, 0]) <= 1e-5 * ref_var[0, 0] + 1e-12
