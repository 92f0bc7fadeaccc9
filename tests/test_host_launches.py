"""What the library decides on the host: the sizes it takes and what it launches, checked without
a GPU against a recording stand-in for the HIP runtime (hip_recorder.cpp).  Each test runs in a
process of its own, where the stand-in's symbols come before the runtime's."""

import ctypes
import importlib.util
import os
import shutil
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

import synth  # noqa: E402


class Lib:
    """libwfs.so over the recording runtime (loaded without the package, which imports torch)."""

    def __init__(self, recorder):
        self.rec = ctypes.CDLL(recorder, mode=ctypes.RTLD_GLOBAL)
        self.rec.rec_take.restype = ctypes.c_char_p
        spec = importlib.util.spec_from_file_location(
            "wfs_ctypes", os.path.join(ROOT, "paper_1608_00386_amd", "_lib.py"))
        self.t = importlib.util.module_from_spec(spec)
        spec.loader.exec_module(self.t)
        self.lib = self.t.lib()

    def set(self, device=0, capturing=0, refuse_attr=0):
        self.rec.rec_set(device, capturing, refuse_attr)

    def lines(self, what):
        """The lines of one kind since the last call: [[name, a, b], ...]."""
        got = [ln.split() for ln in self.rec.rec_take().decode().splitlines()]
        return [ln[1:] for ln in got if ln[0] == what]

    def ops(self):
        """Launches, event records and waits since the last call, in order."""
        got = [ln.split() for ln in self.rec.rec_take().decode().splitlines()]
        return [(ln[0], ln[1], int(ln[2]), int(ln[3])) for ln in got
                if ln[0] in ("on", "record", "wait")]

    def plan(self, cfg, flags=0, batch=1):
        ld = [self.t.layer_desc(x) for x in cfg["layers"]]
        sd = [self.t.sensor_desc(x) for x in cfg["sensors"]]
        h = ctypes.c_void_p()
        rc = self.lib.wfs_plan((self.t.LayerDesc * len(ld))(*ld), len(ld), cfg["layer_stride"],
                               (self.t.SensorDesc * len(sd))(*sd), len(sd), batch,
                               cfg["lambda_ref_m"], cfg["dt_s"], flags, ctypes.byref(h))
        assert rc == 0, self.lib.wfs_last_error()
        return h

    def adjoint(self, plan):
        fake = ctypes.c_void_p(4096)  # (kernels are not run)
        return self.lib.wfs_adjoint(plan, fake, fake, None, None, 0, fake, None)


def _case(n_sub, layers, n_pix):
    bin_ = next(b for b in range(1, 99) if b * n_pix >= 2 * n_sub and b * n_pix % 2 == 0)
    return synth.small_lgs(n_sa=3, n_sub=n_sub, n_fft=n_pix * bin_, bin_=bin_, n_layers=layers,
                           n=32, pitch=0.5)


# (n_sub, layers, image pixels): sizes whose spot waves fit 64 KB of LDS a workgroup with room
# for the adjoint's lag classes: many layers, the largest images, images of one pixel (every lag
# in a class), with the stencil taps in the same LDS (atomic form) or not
ADJOINT = [(12, 18, 12, False), (12, 24, 12, False), (12, 20, 12, False), (10, 24, 14, False),
           (10, 30, 10, False), (10, 31, 8, False), (10, 43, 8, False), (12, 33, 9, False),
           (4, 64, 19, False), (12, 17, 1, False), (12, 22, 1, False), (12, 17, 1, True),
           (12, 19, 1, True), (9, 38, 1, True), (12, 18, 5, True)]


def child_adjoint_sizes(L):
    for n_sub, layers, n_pix, atomic in ADJOINT:
        h = L.plan(_case(n_sub, layers, n_pix),
                   L.t.WFS_FLAG_ADJOINT_ATOMIC if atomic else 0)
        assert L.adjoint(h) == 0, (n_sub, layers, n_pix, atomic, L.lib.wfs_last_error())
        assert L.lib.wfs_plan_destroy(h) == 0
        assert not L.lines("refused")


def child_adjoint_clear(L):
    """A clear recorded into a graph is no clear yet: the graph may never be launched."""
    for warm in (False, True):  # whether an eager call comes before the capture
        h = L.plan(_case(4, 2, 4))
        L.lines("launch")
        cleared = []
        for capturing in ([0] if warm else []) + [1, 1, 0, 0, 1]:
            L.set(capturing=capturing)
            assert L.adjoint(h) == 0, L.lib.wfs_last_error()
            cleared.append(sum("zero_kernel" in name for name, _, _ in L.lines("launch")))
        assert cleared == ([1, 0, 0, 0, 0, 0] if warm else [1, 1, 1, 0, 0]), cleared
        assert L.lib.wfs_plan_destroy(h) == 0


def child_lds_of_every_device(L):
    """Kernels with more than 64 KB of LDS, on two devices of one process; a refused attribute is
    an error of that call only."""
    fake = ctypes.c_void_p(4096)
    big = _case(4, 2, 4)
    big["sensors"].append(synth.configs._ngs(theta_x=0.0, theta_y=0.0, n_sa=1, n_sub=40,
                                             n_fft=128, bin_=4, lam=1.65e-6, photons=0.0,
                                             read_noise=0.0, pupil_d=6.0, obs_d=1.0))

    def screen(n):
        return L.lib.screen_generate(n, 0.1, 0.1, 25.0, 1, 0, fake, fake, 2 * n * n, None)

    for device in (0, 1, 0):
        L.set(device=device, refuse_attr=1)
        assert screen(4096) != 0
        L.set(device=device)
        for n in (1024, 2048, 4096):
            assert screen(n) == 0, (device, n, L.lib.wfs_last_error())
        h = L.plan(big)
        assert L.lib.wfs_forward(h, fake, 0, 42, fake, None, None) == 0, L.lib.wfs_last_error()
        names = L.lines("launch")
        assert any("fft_spot_kernel" in n and int(lds) > 65536 for n, _, lds in names), names
        assert L.lib.wfs_plan_destroy(h) == 0


def _unjoined(lines, caller=0):
    """Streams with work that the caller's stream does not wait for: `seen[s]` holds how many
    launches of every stream the work of stream s comes after."""
    count, seen, events = {}, {}, {}
    for ln in lines:
        kind, _, a, b = ln
        if kind == "on":
            count[a] = count.get(a, 0) + 1
            seen.setdefault(a, {})[a] = count[a]
        elif kind == "record":
            events[b] = dict(seen.get(a, {}))
        elif kind == "wait":
            mine = seen.setdefault(a, {})
            for k, v in events.get(b, {}).items():
                mine[k] = max(mine.get(k, 0), v)
    return [s for s, n in count.items() if seen.get(caller, {}).get(s, 0) < n]


def child_second_streams(L):
    """Whatever launch fails, the work that got as far as a second stream is waited for by the
    caller's stream, whose owner may free the buffers after an error."""
    fake = ctypes.c_void_p(4096)
    cfg = _case(4, 2, 4)
    cfg["sensors"].append(synth.configs._ngs(theta_x=0.0, theta_y=0.0, n_sa=1, n_sub=40,
                                             n_fft=128, bin_=4, lam=1.65e-6, photons=0.0,
                                             read_noise=0.0, pupil_d=6.0, obs_d=1.0))
    cfg["layers"].append(dict(nx=8, ny=8, pitch_m=1.0, alt_m=0.0, vx_mps=0.0, vy_mps=0.0,
                              weight=-1.0, boundary=1))
    o = cfg["layers"][-1]["offset"] = cfg["layer_stride"]
    cfg["layer_stride"] += 64
    h = L.plan(cfg, batch=4)
    n = ctypes.c_int64()
    assert L.lib.wfs_calibrate_work(h, ctypes.byref(n)) == 0
    work = (ctypes.c_float * n.value)()
    calls = {"forward": lambda: L.lib.wfs_forward(h, fake, 0, 42, fake, None, None),
             "calibrate": lambda: L.lib.wfs_calibrate(h, fake, o, 8, 0.1, 0, 42, fake, 1 << 20,
                                                      None, work, n.value, None)}
    for frames in range(4):
        def steps(frames=frames):
            assert L.lib.wfs_plan_set_schedule(h, -1, frames, -1, -1, -1, -1) == 0
            return L.lib.wfs_forward_steps(h, fake, 0, 4, 42, fake, None, None)
        calls["steps%d" % frames] = steps
    for name, call in calls.items():
        L.ops()
        assert call() == 0, (name, L.lib.wfs_last_error())
        ops = L.ops()
        launches = sum(x[0] == "on" for x in ops)
        assert launches > 2 and any(x[0] == "wait" for x in ops), (name, launches)
        assert not _unjoined(ops), name
        for i in range(launches):
            L.rec.rec_fail_launch(i)
            assert call() == L.t.WFS_EDEVICE, (name, i)
            assert not _unjoined(L.ops()), (name, i, "of", launches)
    L.rec.rec_fail_launch(-1)


def _run(case, tmp_path):
    import pytest
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    so = str(tmp_path / "hip_recorder.so")
    src = os.path.join(ROOT, "tests", "hip_recorder.cpp")
    subprocess.run([cxx, "-std=c++17", "-O1", "-shared", "-fPIC", src, "-o", so], check=True)
    r = subprocess.run([sys.executable, os.path.abspath(__file__), case, so],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr


def test_adjoint_takes_every_size_that_fits_its_lds(tmp_path):
    _run("adjoint_sizes", tmp_path)


def test_adjoint_clears_its_images_outside_a_capture(tmp_path):
    _run("adjoint_clear", tmp_path)


def test_large_lds_is_allowed_on_every_device(tmp_path):
    _run("lds_of_every_device", tmp_path)


def test_second_streams_are_joined_whatever_fails(tmp_path):
    _run("second_streams", tmp_path)


if __name__ == "__main__":
    globals()["child_" + sys.argv[1]](Lib(sys.argv[2]))
