"""The library's stream ordering against a model of the HIP runtime with several
devices (tests/hip_model.c), in a process of its own without torch."""
import ctypes as C
import importlib.util
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("hip") / "libhip_model.so")
    subprocess.run(["gcc", "-O1", "-std=c11", "-fPIC", "-shared", "-Wall",
                    os.path.join(ROOT, "tests", "hip_model.c"), "-o", out], check=True)
    return out


def run_case(model, name):
    r = subprocess.run([sys.executable, os.path.abspath(__file__), model, name],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr


class Log:
    """The model's log as operations, each with what has certainly run before it."""

    def __init__(self, text):
        self.ops, count, seen, events = [], {}, {}, {}
        for ln in text.splitlines():
            kind, *f = ln.split()
            if kind == "record":
                s = (int(f[1]), int(f[2]))
                events[f[0]] = {**seen.get(s, {}), s: count.get(s, 0)}
                continue
            s = (int(f[0]), int(f[1]))
            mine = seen.setdefault(s, {})
            if kind == "wait":
                for k, n in events[f[2]].items():
                    mine[k] = max(mine.get(k, 0), n)
                continue
            count[s] = count.get(s, 0) + 1
            self.ops.append((kind, s, count[s], dict(mine), f[2:]))

    def on(self, stream):
        return [o for o in self.ops if o[1] == stream]


def before(a, b):
    return a[2] < b[2] if a[1] == b[1] else b[3].get(a[1], 0) >= a[2]


# ---- in the process of its own ---------------------------------------------
class Bench:
    def __init__(self, model):
        self.hip = C.CDLL(model, mode=C.RTLD_GLOBAL)
        self.hip.model_log.restype = C.c_char_p
        self.hip.model_stream.restype = C.c_void_p
        self.hip.model_id.argtypes = [C.c_void_p]
        spec = importlib.util.spec_from_file_location(
            "abi", os.path.join(ROOT, "paper_2409_07563_amd", "_abi.py"))
        self.abi = importlib.util.module_from_spec(spec)
        spec.loader.exec_module(self.abi)
        self.L, self.keep = self.abi.lib(), []

    def context(self, stream, batch=0, grad=False):
        """A double-integrator context (or a batch of them; grad: a bicycle with
        gradients) on a stream of the model."""
        abi, n = self.abi, max(1, batch)
        cfg, par = (abi.Config * n)(), (abi.Params * n)()
        model = "bicycle" if grad else "double_integrator"
        state = 5 if grad else 4
        ref = (C.c_float * (5 * 21))()
        for c, p in zip(cfg, par):
            c.abi_version = abi.ABI_VERSION
            c.dynamics, c.cost = abi.DYNAMICS[model], abi.COSTS["track" if grad else "quadratic"]
            c.integrator = abi.INTEGRATORS["rk4" if grad else "euler"]
            c.num_samples, c.horizon, c.state_dim, c.control_dim = 100, 20, state, 2
            c.dt, c.lam = 0.1, 1.0
            c.sigma[0] = c.sigma[1] = 1.0
            c.flags = abi.F_REQUIRES_GRAD if grad else 0
            p.wheelbase, p.ref, p.ref_len = 2.5, ref, len(ref)
        size = (self.L.mppi_batch_workspace_bytes(cfg, par, n) if batch
                else self.L.mppi_workspace_bytes(cfg, par))
        assert size, self.L.mppi_last_error()
        ws = C.create_string_buffer(size + 256)
        at = (C.addressof(ws) + 255) // 256 * 256
        self.keep += [cfg, par, ref, ws]
        ctx = C.c_void_p()
        if batch:
            self.ok(self.L.mppi_create_batch(cfg, par, n, at, size, stream, C.byref(ctx)))
        else:
            self.ok(self.L.mppi_create(cfg, par, at, size, stream, C.byref(ctx)))
        self.floats = C.create_string_buffer(1 << 20)
        self.hip.model_clear()
        return ctx

    def ok(self, status):
        assert status == 0, self.L.mppi_last_error()

    def log(self):
        return Log(self.hip.model_log().decode())

    def work(self, dev, stream=None):
        """An operation of the caller's on one of its streams."""
        cur = self.hip.model_current()
        self.hip.hipSetDevice(dev)
        self.hip.hipMemsetAsync(None, 0, C.c_size_t(0), C.c_void_p(stream))
        self.hip.hipSetDevice(cur)

    def mark(self):
        return len(self.log().ops)


def case_other_device(b):
    """A context of device 1 while device 0 is current: the null stream it is
    ordered with is device 1's, and so are its events."""
    s = b.hip.model_stream(1)
    ctx = b.context(s)
    lib = (1, b.hip.model_id(s))
    b.work(1)                                    # the caller writes a state
    b.ok(b.L.mppi_wait_stream(ctx, None))
    b.ok(b.L.mppi_set_state(ctx, b.floats))
    b.ok(b.L.mppi_release_stream(ctx, None))
    b.work(1)                                    # and uses a result
    log = b.log()
    first, last = log.on((1, 0))
    copy = log.on(lib)[0]
    assert before(first, copy) and before(copy, last)
    assert b.hip.model_current() == 0


def case_other_device_stream(b):
    """The same with a stream of its own that the caller makes there."""
    s, mine = b.hip.model_stream(1), b.hip.model_stream(1)
    ctx = b.context(s)
    b.work(1, mine)
    b.ok(b.L.mppi_wait_stream(ctx, mine))
    b.ok(b.L.mppi_set_state(ctx, b.floats))
    b.ok(b.L.mppi_release_stream(ctx, mine))
    b.work(1, mine)
    log = b.log()
    first, last = log.on((1, b.hip.model_id(mine)))
    copy = log.on((1, b.hip.model_id(s)))[0]
    assert before(first, copy) and before(copy, last)


CASES = {n[5:]: f for n, f in list(globals().items()) if n.startswith("case_")}


@pytest.mark.parametrize("name", sorted(CASES))
def test_ordering(model, name):
    run_case(model, name)


if __name__ == "__main__":
    CASES[sys.argv[2]](Bench(sys.argv[1]))
