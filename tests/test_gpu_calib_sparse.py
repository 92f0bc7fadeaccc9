"""wfs_calibrate on noise-free sensors and mirror actuators forms only the subapertures a poke
can reach; the rows are those of the dense batch bit for bit.  WFS_FLAG_SPLIT keeps a plan on
the dense batch (its sensors stage no footprint), so the two are compared over the forms the
call takes: several mirrors, padding elements, subaperture sizes, FFT-path sensors, on-sky
screens with wind, sodium profiles, batch sizes and non-finite screens."""

import copy

import numpy as np
import pytest

import synth
from test_oracle_calib import _system
from wfs_cases import dm_case, mixed_case, uneven_case

pytestmark = pytest.mark.gpu


def _gpu():
    import torch
    import paper_1608_00386_amd as W
    return torch, W


def _quiet(cfg):
    cfg = copy.deepcopy(cfg)
    for s in cfg["sensors"]:
        s["photons"] = s["read_noise_e"] = 0.0
    return cfg


def _with_mirrors(cfg, grids, pad=0):
    """Mirror grids (n, pitch, altitude) after the layers; ``pad`` elements between them."""
    cfg = _quiet(cfg)
    offs, stride = synth.layer_offsets(cfg["layers"])
    for L, o in zip(cfg["layers"], offs):
        L["offset"] = o
    first = stride
    for nx, ny, pitch, alt in grids:
        cfg["layers"].append(dict(offset=stride, nx=nx, ny=ny, pitch_m=pitch, alt_m=alt,
                                  vx_mps=0.0, vy_mps=0.0, weight=-1.0, boundary=1, r0_m=None,
                                  L0_m=None))
        stride += nx * ny + pad
    cfg["layer_stride"] = (stride + 3) // 4 * 4
    return cfg, first, stride - first


def _case(name):
    """(config, first actuator, actuators, step, base kind)."""
    if name == "dm7":
        cfg, a0, n = _system()
        return dict(cfg, batch=8), a0, n, 0, None
    if name == "dm7_onsky_wind":
        cfg, a0, n = _system(turbulence=True, wind=(35.0, -20.0))
        return dict(cfg, batch=6), a0, n, 11, "screen"
    if name == "two_ngs_dm11_layers":
        cfg = _quiet(dm_case())
        L = cfg["layers"][-1]
        return dict(cfg, batch=4), L["offset"], L["nx"] * L["ny"], 5, "screen"
    if name == "mixed_fft":  # an FFT-path sensor; mirrors finer and coarser than subapertures
        cfg, a0, n = _with_mirrors(mixed_case(), [(9, 8, 0.8, 0.0), (21, 19, 0.35, 3000.0)], pad=5)
        return dict(cfg, batch=10), a0, n, 2, "screen"
    if name == "uneven_fft":
        cfg, a0, n = _with_mirrors(uneven_case(), [(16, 16, 1.0, 500.0)])
        return dict(cfg, batch=12), a0 + 7, n - 20, 3, "screen"
    if name == "nan_screen":
        cfg, a0, n = _with_mirrors(uneven_case(fft=False), [(16, 16, 1.0, 500.0)])
        return dict(cfg, batch=4), a0, n, 1, "nan"
    if name == "tiny_mirror_pitch":  # many actuators per pixel: most pokes reach nothing
        cfg, a0, n = _with_mirrors(mixed_case(), [(24, 24, 0.05, 0.0)])
        return dict(cfg, batch=16), a0, n, 0, None
    raise KeyError(name)


@pytest.mark.parametrize("name", ["dm7", "dm7_onsky_wind", "two_ngs_dm11_layers", "mixed_fft",
                                  "uneven_fft", "nan_screen", "tiny_mirror_pitch"])
def test_sparse_rows_equal_the_dense_batch(name):
    torch, W = _gpu()
    cfg, a0, n, step, kind = _case(name)
    base = None
    if kind:
        b = np.random.default_rng(4).standard_normal(cfg["layer_stride"]) * 0.4
        if kind == "nan":
            b[3 * cfg["layers"][0]["nx"] + 40] = np.nan
            b[a0 + 9] = np.inf
        base = torch.from_numpy(b.astype(np.float32)).cuda()
    if any(s["na_fwhm_m"] > 0 for s in cfg["sensors"]) and name != "dm7":
        cfg = dict(cfg, na_profile=[[(0.0, 9e3, 1.0)], [(-4e3, 3e3, 2.0), (5e3, 0.0, 1.0)]])
    dense = W.Plan(cfg, flags=W.WFS_FLAG_SPLIT)
    want, want_ref = dense.calibrate(a0, n, amplitude=-0.4, step=step, base=base)
    for batch in (cfg["batch"], 2):
        plan = W.Plan(cfg, batch=batch)
        fill = torch.full((n, plan.n_slopes + 3), 5.0, device="cuda")
        got, ref = plan.calibrate(a0, n, amplitude=-0.4, step=step, base=base, im=fill)
        assert torch.equal(ref.view(torch.int32), want_ref.view(torch.int32))
        assert torch.equal(got[:, :plan.n_slopes].contiguous().view(torch.int32),
                           want.view(torch.int32))
        assert torch.all(got[:, plan.n_slopes:] == 5.0)
    if name not in ("nan_screen", "tiny_mirror_pitch"):  # some rows are not zero
        assert float(want.abs().max()) > 1e-3


def test_sparse_calibration_replays_in_a_graph():
    torch, W = _gpu()
    cfg, a0, n, step, _ = _case("mixed_fft")
    plan = W.Plan(cfg)
    base = torch.randn(cfg["layer_stride"], device="cuda") * 0.3
    im = torch.empty(n, plan.n_slopes, device="cuda")
    plan.calibrate(a0, n, amplitude=0.3, step=step, base=base, im=im)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        plan.calibrate(a0, n, amplitude=0.3, step=step, base=base, im=im)
    for k in range(3):
        base.copy_(torch.randn(cfg["layer_stride"], device="cuda") * 0.3)
        im.zero_()
        graph.replay()
        torch.cuda.synchronize()
        got = im.clone()
        want, _ = plan.calibrate(a0, n, amplitude=0.3, step=step, base=base)
        assert torch.equal(got, want), k
