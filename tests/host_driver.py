"""Runs the library's host code against tests/hip_double.c, in a process of its
own without torch (which would bring the real runtime along):

    python tests/host_driver.py <double.so> <check> [<JSON argument>]

prints the check's result as JSON."""
import ctypes as C
import importlib.util
import json
import math
import os
import subprocess
import sys
import tempfile

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
from synth import scene as S  # noqa: E402


def check(tmp_path_factory, name, arg=None):
    """The result of a check, from a test."""
    out = tmp_path_factory.getbasetemp() / "hip_double.so"
    if not out.exists():
        subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                        os.path.join(ROOT, "tests", "hip_double.c"), "-o", str(out)], check=True)
    env = dict(os.environ)
    env.setdefault("PSFS_AUTOTUNE_CACHE", os.path.join(tempfile.mkdtemp(dir=tmp_path_factory.getbasetemp()), "tune.json"))
    r = subprocess.run([sys.executable, os.path.abspath(__file__), str(out), name, json.dumps(arg)],
                       capture_output=True, text=True, timeout=120, env=env)
    assert r.returncode == 0, r.stderr[-2000:]
    return json.loads(r.stdout.splitlines()[-1])


def _load(double):
    spec = importlib.util.spec_from_file_location("psfs_signatures", os.path.join(ROOT, "paper_1311_6811_amd", "_lib.py"))
    L = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(L)
    dbl = C.CDLL(double, mode=C.RTLD_GLOBAL)
    dbl.dbl_launch.restype, dbl.dbl_cost.argtypes = C.c_char_p, [C.c_char_p, C.c_float]
    return L, L.lib(), dbl


FAKE = 1 << 20                  # a device address that nothing reads


class Host:
    def __init__(self, double):
        self.L, self.lib, self.dbl = _load(double)

    def cameras(self, cams):
        arr = (self.L.psfs_camera * max(len(cams), 1))()
        for a, c in zip(arr, cams):
            a.width, a.height, a.P = c.width, c.height, tuple(np.asarray(c.P, np.float32).reshape(12).tolist())
        return arr

    def grid(self, nx, ny, nz, side=2.0):
        h = np.float32(side / max(nx, ny, nz))
        return self.L.psfs_grid(nx, ny, nz, tuple(float(np.float32(-0.5 * h * d)) for d in (nx, ny, nz)), float(h))

    def params(self, sampling=0):
        return self.L.psfs_params(0.5, -3.0 * math.log(256.0), 0.5, sampling)

    def plan(self, cams, grid, sampling=0, backgrounds=True):
        h = C.c_void_p()
        assert self.lib.psfs_plan_create(C.byref(h)) == 0
        assert self.lib.psfs_set_cameras(h, len(cams), self.cameras(cams)) == 0
        assert self.lib.psfs_set_grid(h, C.byref(grid)) == 0
        assert self.lib.psfs_set_params(h, C.byref(self.params(sampling))) == 0
        for k in range(len(cams) if backgrounds else 0):
            assert self.lib.psfs_set_background(h, k, FAKE, FAKE) == 0
        return h

    def fakes(self, n):
        return self.L.ptr_array([FAKE] * n)

    def launches(self):
        """[(kernel, grid, workgroup)] since the last look."""
        out = []
        for k in range(self.dbl.dbl_launches()):
            dim = (C.c_uint * 6)()
            name = self.dbl.dbl_launch(k, dim).decode()
            out.append((name, list(dim[:3]), list(dim[3:])))
        self.dbl.dbl_reset()
        return out


def diff_forward_at(host, arg):
    """psfs_diff_forward_at with a failing runtime: the status, copies still under
    way at its return and whether the plan had taken the views (its likelihood
    then finds backgrounds)."""
    cams = S.ring_rig(2, 100.0, 32, 24)
    plan = host.plan(cams, host.grid(8, 8, 8), 1, backgrounds=False)
    P = np.stack([np.asarray(c.P, np.float32) + 1 for c in cams]).astype(np.float32)
    ws = host.lib.psfs_diff_workspace_bytes(plan)
    bg, ims = host.fakes(2), host.fakes(2)
    if arg["fail"] == "record":
        host.dbl.dbl_fail_record(1)
    elif arg["fail"]:
        host.dbl.dbl_fail_launch(arg["fail"])
    taken = host.cameras(cams)
    rc = host.lib.psfs_diff_forward_at(plan, 2, taken, P.ctypes.data, bg, bg, ims, FAKE, None, FAKE, FAKE, FAKE, ws, None)
    pending = host.dbl.dbl_pending()
    host.dbl.dbl_reset()
    ready = host.lib.psfs_likelihood(plan, ims, FAKE, None) == 0
    got = [list(c.P) for c in taken] == P.reshape(2, 12).tolist()
    host.lib.psfs_plan_destroy(plan)
    return dict(rc=rc, pending=pending, ready=ready, matrices=got)


def fusion_kernels(host, arg):
    """The kernel that psfs_fuse launches on every tile (-1 too), and the tile
    that psfs_get_tile then reports."""
    cams = S.ring_rig(arg["n"], 0.9375 * arg["W"], arg["W"], arg["H"])
    plan = host.plan(cams, host.grid(*arg["grid"]), arg["sampling"])
    out = []
    for tile in range(-1, host.lib.psfs_tile_count()):
        assert host.lib.psfs_set_tile(plan, tile) == 0
        reported = host.lib.psfs_get_tile(plan)
        host.launches()
        assert host.lib.psfs_fuse(plan, FAKE, FAKE, FAKE, None) == 0
        (name, grid, group), = host.launches()
        out.append((tile, reported, name, grid, group))
    host.lib.psfs_plan_destroy(plan)
    return out


def surface_launches(host, arg):
    """Kernels of psfs_surface with their grids and workgroups."""
    plan = host.plan([], host.grid(*arg["grid"]), 0)
    nbytes = host.lib.psfs_surface_workspace_bytes(plan)
    host.launches()
    assert host.lib.psfs_surface(plan, FAKE, FAKE, FAKE, FAKE, 8, FAKE, FAKE, nbytes, None) == 0
    return host.launches()


def inside(host, arg):
    """For random rigs and grids: what the host says of "the whole grid is inside
    the view", and what FP32 projections of every voxel centre say, as the kernels
    form them. Returns [said, and how many centres fall outside]."""
    class ViewGeom(C.Structure):
        _fields_ = [("P", C.c_float * 12), ("W", C.c_int32), ("H", C.c_int32), ("map_off", C.c_int64)]
    f = host.lib._ZN4psfs4host11grid_insideERKNS_8ViewGeomERK9psfs_grid
    f.restype = C.c_bool
    rng = np.random.default_rng(arg["seed"])
    out = []
    for _ in range(arg["count"]):
        dims = rng.integers(1, 40, 3)
        grid = host.grid(*[int(d) for d in dims], side=float(rng.uniform(0.5, 6.0)))
        W, H = (int(x) for x in rng.choice([(320, 240), (641, 479), (65535, 900)]))
        cam = S.ring_rig(8, 0.9375 * W * rng.uniform(0.5, 1.5), W, H, float(rng.uniform(1.5, 6.0)))[int(rng.integers(8))]
        P = np.asarray(cam.P, np.float64).reshape(3, 4)
        P[:2] += 0.5 * P[2]
        g = ViewGeom(tuple(P.astype(np.float32).reshape(12).tolist()), W, H, 0)
        P = np.array(list(g.P), np.float32).reshape(3, 4)
        x, y, z = (np.float32(grid.origin[d]) + np.float32(grid.voxel) * (np.arange(dims[d]).astype(np.float32) + np.float32(0.5))
                   for d in range(3))
        rows = [P[r, 0] * x[None, None, :] + (P[r, 1] * y[None, :, None] + P[r, 3]) + P[r, 2] * z[:, None, None] for r in range(3)]
        with np.errstate(divide="ignore", invalid="ignore"):
            u, v = rows[0] / rows[2], rows[1] / rows[2]
        seen = (rows[2] > 0) & (u >= 0) & (u < W) & (v >= 0) & (v < H)
        out.append((bool(f(C.byref(g), C.byref(grid))), int((~seen).sum())))
    return out


def _sequence(host, plan, n):
    """Kernels of a fusion and of a one-frame step."""
    host.launches()
    assert host.lib.psfs_fuse(plan, FAKE, FAKE, FAKE, None) == 0
    assert host.lib.psfs_pipeline_step(plan, host.fakes(n), FAKE, FAKE + (1 << 30), FAKE, None, None) == 0
    return [name for name, _, _ in host.launches()]


def tuned_plan(host, arg):
    """A plan tuned while launches take `costs` [(part of the name, ms)]: the tile
    returned and reported, the kernels it then runs, those of a second plan
    tuned from the cache, and of one that was not tuned; the cache."""
    cams = S.ring_rig(arg["n"], 0.9375 * arg["W"], arg["W"], arg["H"])
    out = {}
    if arg.get("cache"):
        with open(os.environ["PSFS_AUTOTUNE_CACHE"], "w") as f:
            json.dump(arg["cache"], f)
    for name in ("timed", "cached", "untuned"):
        plan = host.plan(cams, host.grid(*arg["grid"]), arg["sampling"])
        best = C.c_int32(-1)
        if name != "untuned":
            for part, ms in arg["costs"] if name == "timed" else []:
                host.dbl.dbl_cost(part.encode(), ms)
            ws = host.lib.psfs_tune_workspace_bytes(plan) + (0 if arg.get("short") else host.lib.psfs_workspace_bytes(plan))
            rc = host.lib.psfs_tune(plan, host.fakes(arg["n"]), FAKE, ws, None, 0, C.byref(best))
            assert rc == 0, host.lib.psfs_last_error()
        launched = len(host.launches())
        out[name] = dict(best=best.value, reported=host.lib.psfs_get_tile(plan), launched=launched,
                         kernels=_sequence(host, plan, arg["n"]))
        host.lib.psfs_plan_destroy(plan)
    with open(os.environ["PSFS_AUTOTUNE_CACHE"]) as f:
        out["cache"] = json.load(f)
    return out


def _batch(host, arg):
    frames = [(S.ring_rig(n, 0.9375 * W, W, H), host.grid(*grid)) for grid, n, W, H in arg["frames"]]
    arr = (host.L.psfs_frame * len(frames))()
    keep = []
    for a, (cams, grid) in zip(arr, frames):
        keep += [host.cameras(cams), host.fakes(len(cams))]
        a.grid, a.n, a.cams = grid, len(cams), keep[-2]
        a.images_dev = a.mean_dev = a.var_dev = keep[-1]
        a.posterior_dev = FAKE
    h = C.c_void_p()
    assert host.lib.psfs_batch_create(C.byref(h), C.byref(host.params(arg["sampling"])), len(frames), arr) == 0
    return h, arr, keep


def tuned_batch(host, arg):
    """As tuned_plan, for a batch; the kernels are those of a run."""
    out = {}
    if arg.get("cache"):
        with open(os.environ["PSFS_AUTOTUNE_CACHE"], "w") as f:
            json.dump(arg["cache"], f)
    for name in ("timed", "cached", "untuned"):
        h, _, _ = _batch(host, arg)
        nbytes = host.lib.psfs_batch_workspace_bytes(h)
        best = C.c_int32(-1)
        if name != "untuned":
            for part, ms in arg["costs"] if name == "timed" else []:
                host.dbl.dbl_cost(part.encode(), ms)
            assert host.lib.psfs_batch_tune(h, FAKE, nbytes, None, 0, C.byref(best)) == 0
        launched = len(host.launches())
        assert host.lib.psfs_batch_run(h, FAKE, nbytes, None) == 0
        out[name] = dict(best=best.value, reported=host.lib.psfs_batch_get_tile(h), launched=launched,
                         kernels=[k for k, _, _ in host.launches()])
        host.lib.psfs_batch_destroy(h)
    with open(os.environ["PSFS_AUTOTUNE_CACHE"]) as f:
        out["cache"] = json.load(f)
    return out


def batch_kernels(host, arg):
    """Of a batch of these frames (grid, views, image size) on every tile (-1
    too): the tile that psfs_batch_get_tile reports, the kernels of a run and of
    the run after a same-shape update."""
    h, arr, _keep = _batch(host, arg)
    nbytes = host.lib.psfs_batch_workspace_bytes(h)
    out = []
    for tile in arg.get("tiles") or [*range(-1, host.lib.psfs_tile_count()), -1]:
        assert host.lib.psfs_batch_set_tile(h, tile) == 0
        runs = []
        for _ in range(2):
            host.launches()
            assert host.lib.psfs_batch_run(h, FAKE, nbytes, None) == 0
            runs.append(host.launches())
            assert host.lib.psfs_batch_update(h, len(arr), arr) == 0
        out.append((tile, host.lib.psfs_batch_get_tile(h), *runs))
    host.lib.psfs_batch_destroy(h)
    return out


if __name__ == "__main__":
    print(json.dumps(globals()[sys.argv[2]](Host(sys.argv[1]), json.loads(sys.argv[3]))))
