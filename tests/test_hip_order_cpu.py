"""The library's stream ordering and the grids of its largest launches against a model of the HIP runtime with several
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
        self.floats = C.create_string_buffer(1 << 20)

    def context(self, stream, batch=0, grad=False, hidden=0, bf16=False, K=100):
        """A double-integrator context (or a batch of them; hidden: a bicycle with an
        MLP residual, grad: a bicycle with gradients) on a stream of the model."""
        abi, n = self.abi, max(1, batch)
        cfg, par = (abi.Config * n)(), (abi.Params * n)()
        model = "bicycle_mlp" if hidden else "bicycle" if grad else "double_integrator"
        track = bool(grad or hidden)
        state = 5 if track else 4
        ref = (C.c_float * (5 * 21))()
        mlp = (C.c_float * (14 * hidden + hidden**2 + 5))()
        for c, p in zip(cfg, par):
            c.abi_version = abi.ABI_VERSION
            c.dynamics, c.cost = abi.DYNAMICS[model], abi.COSTS["track" if track else "quadratic"]
            c.integrator = abi.INTEGRATORS["rk4" if track else "euler"]
            c.num_samples, c.horizon, c.state_dim, c.control_dim = K, 20, state, 2
            c.dt, c.lam = 0.1, 1.0
            c.sigma[0] = c.sigma[1] = 1.0
            c.flags = (abi.F_REQUIRES_GRAD if grad else 0) | (abi.F_BF16_MLP if bf16 else 0)
            p.mlp_hidden, p.mlp = hidden, mlp
            p.wheelbase, p.ref, p.ref_len = 2.5, ref, len(ref)
        size = (self.L.mppi_batch_workspace_bytes(cfg, par, n) if batch
                else self.L.mppi_workspace_bytes(cfg, par))
        assert size, self.L.mppi_last_error()
        ws = C.create_string_buffer(size + 256)
        at = (C.addressof(ws) + 255) // 256 * 256
        self.keep = [cfg, par, ref, mlp, ws]
        ctx = C.c_void_p()
        if batch:
            self.ok(self.L.mppi_create_batch(cfg, par, n, at, size, stream, C.byref(ctx)))
        else:
            self.ok(self.L.mppi_create(cfg, par, at, size, stream, C.byref(ctx)))
        self.hip.model_clear()
        return ctx

    def bicycle(self, K, T, cost, flags=0):
        """A bicycle (RK4) context on a stream of the model; cost: "quadratic",
        "circles" (none: "no_circles"), "map" (two values; more: "values"), "goal"."""
        abi = self.abi
        cfg, p = abi.Config(), abi.Params()
        cfg.abi_version, cfg.dynamics = abi.ABI_VERSION, abi.DYNAMICS["bicycle"]
        cfg.cost = abi.COSTS[{"quadratic": "quadratic", "circles": "path_circles",
                              "no_circles": "path_circles", "map": "path_costmap",
                              "values": "path_costmap", "goal": "goal_circles"}[cost]]
        cfg.integrator = abi.INTEGRATORS["rk4"]
        cfg.num_samples, cfg.horizon, cfg.state_dim, cfg.control_dim = K, T, 5, 2
        cfg.dt, cfg.lam = 0.1, 1.0
        cfg.sigma[0] = cfg.sigma[1] = 1.0
        cfg.flags = flags
        four = (C.c_float * 4)(1.0, 2.0, 3.0, 4.0)
        ref = (C.c_float * 5)()
        cells = (C.c_float * 64)(*[float(i if cost == "values" else i % 2) for i in range(64)])
        p.wheelbase, p.ref, p.ref_len = 2.5, ref, 5
        p.num_segments, p.knots, p.coef = 1, four, four
        p.num_circles = 0 if cost == "no_circles" else 2
        p.cx = p.cy = p.r2 = four
        p.map_w = p.map_h = 8
        p.map_res, p.costmap = 1.0, cells
        size = self.L.mppi_workspace_bytes(cfg, p)
        assert size, self.L.mppi_last_error()
        ws = C.create_string_buffer(size + 256) if size < 1 << 28 else None
        # the model runs nothing, so a large workspace is only an address
        at = (C.addressof(ws) + 255) // 256 * 256 if ws else 1 << 40
        self.keep = [cfg, p, four, ref, cells, ws]
        ctx = C.c_void_p()
        self.ok(self.L.mppi_create(cfg, p, at, size, self.hip.model_stream(0), C.byref(ctx)))
        self.ok(self.L.mppi_set_state(ctx, self.floats))
        self.ok(self.L.mppi_sample(ctx))
        return ctx

    def rollout_kernel(self, ctx):
        """(kernel, lanes of the time-parallel form, threads) of the next rollout."""
        n = self.mark()
        self.ok(self.L.mppi_rollout(ctx))
        f = self.log().ops[n][4]
        name = f[4]
        if "rollout_bicycle_scan_kernel" in name:
            return "scan", int(name.split("Li")[-1].split("E")[0]), int(f[3])
        if "rollout_bicycle_group_kernel" in name:
            return "group", int(name.split("Li")[-1].split("E")[0]), int(f[3])
        assert "rollout_kernel" in name, name
        return "lane", 1, int(f[3])

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


def case_put(b):
    """mppi_put reads on the caller's stream, after the context's work and before
    what either stream is given next; on any stream, of any device."""
    for dev, mine in ((0, None), (0, b.hip.model_stream(0)), (1, None), (1, b.hip.model_stream(1))):
        s = b.hip.model_stream(dev)
        ctx = b.context(s)
        lib, cur = (dev, b.hip.model_id(s)), (dev, b.hip.model_id(mine))
        for what in (b.abi.PACKED_STATE, b.abi.PACKED_CONTROLS, b.abi.PACKED_SAMPLES):
            b.ok(b.L.mppi_sample(ctx))
            n = b.mark()
            b.ok(b.L.mppi_put(ctx, what, b.floats, mine))
            b.ok(b.L.mppi_sample(ctx))
            new = b.log().ops[n:]
            copy = [o for o in new if o[1] == cur]
            assert len(copy) == 1
            assert before(b.log().ops[n - 1], copy[0]) and before(copy[0], new[-1])
            assert new[-1][1] == lib
        b.L.mppi_destroy(ctx)
    assert b.hip.model_current() == 0


# everything that gives a context work
CALLS = {
    "set_state": lambda b, c: b.L.mppi_set_state(c, b.floats),
    "set_controls": lambda b, c: b.L.mppi_set_controls(c, b.floats),
    "set_costs": lambda b, c: b.L.mppi_set_costs(c, b.floats),
    "set_iteration": lambda b, c: b.L.mppi_set_iteration(c, 3),
    "shift": lambda b, c: b.L.mppi_shift(c, 1, 0),
    "sample": lambda b, c: b.L.mppi_sample(c),
    "rollout": lambda b, c: b.L.mppi_rollout(c),
    "update": lambda b, c: b.L.mppi_update(c),
    "iterate": lambda b, c: b.L.mppi_iterate(c, 1),
    "iterate_graph": lambda b, c: b.L.mppi_iterate(c, 3),
    "get_controls": lambda b, c: b.L.mppi_get_controls(c, b.floats),
    "get_costs": lambda b, c: b.L.mppi_get_debug(c, b.abi.DEBUG_COSTS, b.floats),
    "get_noise": lambda b, c: b.L.mppi_get_debug(c, b.abi.DEBUG_NOISE, b.floats),
    "get_weights": lambda b, c: b.L.mppi_get_debug(c, b.abi.DEBUG_WEIGHTS, b.floats),
    "get_stats": lambda b, c: b.L.mppi_get_debug(c, b.abi.DEBUG_STATS, b.floats),
}


def put_follows(b, ctx, lib, names):
    for name in names:
        # the null stream is ordered after the context, then the context gets work
        b.ok(b.L.mppi_release_stream(ctx, None))
        b.ok(CALLS[name](b, ctx))
        work = b.log().on(lib)[-1]
        b.ok(b.L.mppi_put(ctx, b.abi.PACKED_CONTROLS, b.floats, None))
        copy = b.log().on((0, 0))[-1]
        assert before(work, copy), name
        # a second array straight after it need not wait again, but may not race
        b.ok(b.L.mppi_put(ctx, b.abi.PACKED_STATE, b.floats, None))
        assert before(work, b.log().on((0, 0))[-1]), name


def case_put_after_every_call(b):
    s = b.hip.model_stream(0)
    ctx = b.context(s)
    b.ok(b.L.mppi_set_state(ctx, b.floats))
    b.ok(b.L.mppi_sample(ctx))
    b.ok(b.L.mppi_rollout(ctx))
    put_follows(b, ctx, (0, b.hip.model_id(s)), CALLS)


def case_put_after_every_call_of_a_batch(b):
    s = b.hip.model_stream(0)
    ctx = b.context(s, batch=3)
    b.ok(b.L.mppi_set_state(ctx, b.floats))
    b.ok(b.L.mppi_sample(ctx))
    b.ok(b.L.mppi_rollout(ctx))
    put_follows(b, ctx, (0, b.hip.model_id(s)), CALLS)


def case_put_with_gradients(b):
    s = b.hip.model_stream(0)
    ctx = b.context(s, grad=True)
    lib = (0, b.hip.model_id(s))
    b.ok(b.L.mppi_set_state(ctx, b.floats))
    put_follows(b, ctx, lib, ["sample", "rollout", "update", "iterate"])
    b.ok(b.L.mppi_iterate(ctx, 1))
    for call in (lambda: b.L.mppi_backward(ctx, b.floats, b.floats),
                 lambda: b.L.mppi_set_theta(ctx, (C.c_float * 6)(*[1.0] * 6))):
        b.ok(b.L.mppi_release_stream(ctx, None))
        b.ok(call())
        work = b.log().on(lib)[-1]
        b.ok(b.L.mppi_put(ctx, b.abi.PACKED_CONTROLS, b.floats, None))
        assert before(work, b.log().on((0, 0))[-1])


def case_put_from_two_streams(b):
    """The null stream, then another: each copy follows the one before."""
    s, mine = b.hip.model_stream(0), b.hip.model_stream(0)
    ctx = b.context(s)
    for a, c in ((None, mine), (mine, None)):
        b.ok(b.L.mppi_put(ctx, b.abi.PACKED_STATE, b.floats, a))
        first = b.log().ops[-1]
        b.ok(b.L.mppi_put(ctx, b.abi.PACKED_STATE, b.floats, c))
        assert before(first, b.log().ops[-1])


def case_put_refuses(b):
    ctx = b.context(b.hip.model_stream(0))
    for what, src in ((b.abi.PACKED_NOISE, b.floats), (7, b.floats), (0, None)):
        assert b.L.mppi_put(ctx, what, src, None) == -1
    assert b.L.mppi_put(None, 0, b.floats, None) == -1
    assert b.mark() == 0


def case_noise_of_most_samples(b):
    """mppi_noise up to the last int32 sample count, whose groups are padded to a
    multiple of 8 (or 1024 samples each): a grid that covers them and that HIP takes."""
    sigma = (C.c_float * 8)(*[1.0] * 8)
    for K in (1, 2047, 2049, 2**20, 2**31 - 4096, 2**31 - 2049, 2**31 - 2047, 2**31 - 1024,
              2**31 - 1022, 2**31 - 256, 2**31 - 4, 2**31 - 1):
        for T in (1, 3):
            for ldk in (K, (K + 63) // 64 * 64):
                n = b.mark()
                b.ok(b.L.mppi_noise(1, 0, 0, K, T, 2, sigma, b.floats, ldk, None))
                _, _, _, _, f = b.log().ops[n]
                gx, threads = int(f[0]), int(f[3])
                per = [256, 1024] if ldk % 4 == 0 else [256]  # samples per workgroup
                assert threads == 256 and gx * threads < 2**32, (K, T, ldk, f)
                assert any(gx * p >= K and (gx - 8) * p < K for p in per), (K, T, ldk, f)
                assert gx * 256 <= 2**31, (K, T, ldk, f)  # samples are counted in int32


def case_noise_of_few_samples(b):
    """The groups that fill up the XCDs are at most a third of the launch's own."""
    sigma = (C.c_float * 8)(*[1.0] * 8)
    for K in [*range(1, 5000, 37), 2048, 2049, 3001, 8192, 10007]:
        n = b.mark()
        b.ok(b.L.mppi_noise(1, 0, 0, K, 40, 2, sigma, b.floats, K, None))
        gx = int(b.log().ops[n][4][0])
        groups = -(-K // 256)
        assert gx == groups or (gx % 8 == 0 and groups < gx <= groups + groups // 3), (K, gx)


def case_mlp_rollout_launches(b):
    """Every 16-sample tile in one launch or another, and never more than two
    workgroups per CU of a single wave (which the SIMDs get unevenly)."""
    s = b.hip.model_stream(0)
    for hidden in (16, 32, 64):
        for bf16 in (False, True):
            for grad in (False, True):
                for K in (1, 17, 4096, 8192, 8193, 12288, 12289, 16384, 16385, 17000, 20481,
                          28673, 65536, 65537):
                    ctx = b.context(s, grad=grad, hidden=hidden, bf16=bf16, K=K)
                    b.ok(b.L.mppi_set_state(ctx, b.floats))
                    b.ok(b.L.mppi_sample(ctx))
                    n = b.mark()
                    b.ok(b.L.mppi_rollout(ctx))
                    tiles, low, high = -(-K // 16), 0, 0
                    launches = [o for o in b.log().ops[n:] if o[0] == "launch"]
                    for _, _, _, _, f in launches:
                        groups, threads = int(f[0]), int(f[3])
                        assert threads != 64 or groups <= 512, (hidden, bf16, K, f)
                        # a split tile has four waves (H = 32) or eight, else a wave each
                        most = threads // 64 if threads < 512 else 1
                        low += groups * (1 if hidden == 32 and threads == 256 else most) - most + 1
                        high += groups * most
                    assert 1 <= len(launches) <= 2 and low <= tiles <= high, (hidden, bf16, K)
                    b.L.mppi_destroy(ctx)


def case_sweep_launches(b):
    """H = 32: the reverse sweep's rows in launches of less than two rounds of four
    tiles per CU, none left out."""
    s = b.hip.model_stream(0)
    for K in (100, 4097, 16384, 32752, 32768, 33000, 65536):
        ctx = b.context(s, grad=True, hidden=32, K=K)
        b.ok(b.L.mppi_set_state(ctx, b.floats))
        b.ok(b.L.mppi_iterate(ctx, 1))
        n = b.mark()
        b.ok(b.L.mppi_backward(ctx, b.floats, b.floats))
        grids = [int(o[4][0]) for o in b.log().ops[n:] if o[0] == "launch" and o[4][3] == "384"]
        tiles = -(-K // 16)
        assert all(g <= 1024 for g in grids) and 2 * sum(grids) >= tiles, (K, grids)
        b.L.mppi_destroy(ctx)


def case_default_rollout(b):
    """Where the time-parallel rollout is the default: with cells to search, and
    further out without."""
    want = {  # (cost, K, T): whether time-parallel
        ("circles", 64, 1): True, ("circles", 8192, 5): False, ("circles", 8192, 6): True,
        ("map", 16384, 16): True, ("goal", 32768, 24): True, ("circles", 65536, 48): True,
        ("circles", 65537, 48): False, ("map", 65537, 64): True, ("goal", 70000, 64): True,
        ("quadratic", 64, 11): False, ("quadratic", 64, 12): True, ("values", 8192, 12): True,
        ("no_circles", 8193, 23): False, ("no_circles", 8193, 24): True,
        ("quadratic", 32768, 24): True, ("quadratic", 32769, 200): False,
        ("values", 57344, 48): True, ("values", 57345, 159): False,
        ("no_circles", 57345, 160): True, ("values", 65537, 250): False,
        ("circles", 512, 257): False,
    }
    for (cost, K, T), scan in want.items():
        ctx = b.bicycle(K, T, cost)
        assert (b.rollout_kernel(ctx)[0] == "scan") == scan, (cost, K, T)
        b.L.mppi_destroy(ctx)


def case_partial_tuning(b):
    """Setting one launch shape leaves the others, the rollout's form among them;
    setting what was reported changes nothing."""
    def get(ctx):
        t = b.abi.Tuning()
        b.ok(b.L.mppi_get_tuning(ctx, C.byref(t)))
        return t

    def put(ctx, **shape):
        t = get(ctx)
        for k, v in shape.items():
            setattr(t, k, v)
        return b.L.mppi_set_tuning(ctx, C.byref(t))

    ctx = b.bicycle(8192, 100, "circles")
    assert get(ctx).rollout_form == 0 and get(ctx).lanes_per_sample == 0
    default = b.rollout_kernel(ctx)
    assert default == ("scan", 16, 256)
    for shape in ({}, {"noise_calls": 2}, {"update_form": 0}, {"rollout_block": 128},
                  {"cost_waves": 4}, {"adjoint_tiles": 3}):
        b.ok(put(ctx, **shape))
        assert b.rollout_kernel(ctx) == default, shape
    assert get(ctx).noise_calls == 2 and get(ctx).update_form == 0
    b.ok(put(ctx, lanes_per_sample=4, rollout_block=64))
    assert b.rollout_kernel(ctx) == ("group", 4, 64)
    b.ok(put(ctx))
    assert b.rollout_kernel(ctx) == ("group", 4, 64)
    b.ok(put(ctx, rollout_form=2, lanes_per_sample=32, rollout_block=128))
    assert b.rollout_kernel(ctx) == ("scan", 32, 128)
    assert put(ctx, lanes_per_sample=0) == -1  # the scan form names its lanes
    b.ok(put(ctx, rollout_form=0, lanes_per_sample=0))
    assert b.rollout_kernel(ctx) == default
    b.ok(put(ctx, rollout_form=1))  # the split form with the fused form's lanes
    assert get(ctx).lanes_per_sample == 4
    b.L.mppi_destroy(ctx)
    for K, cost, kernel in ((40000, "quadratic", ("lane", 1, 256)),
                            (20000, "quadratic", ("group", 4, 64))):
        ctx = b.bicycle(K, 20, cost)
        assert b.rollout_kernel(ctx) == kernel
        assert (get(ctx).lanes_per_sample, get(ctx).rollout_block) == kernel[1:]
        b.ok(put(ctx, noise_calls=4))
        assert b.rollout_kernel(ctx) == kernel
        assert put(ctx, lanes_per_sample=0) == -1  # not the library's choice here
        b.L.mppi_destroy(ctx)
    for flag, kernel in ((b.abi.F_ROLLOUT_LANE, ("lane", 1, 64)), (b.abi.F_ROLLOUT_QUAD, ("group", 4, 64))):
        ctx = b.bicycle(500, 60, "circles", flag)
        assert b.rollout_kernel(ctx) == kernel and get(ctx).lanes_per_sample == kernel[1]
        assert put(ctx, lanes_per_sample=0) == -1
        b.L.mppi_destroy(ctx)
    for make in (lambda: b.context(b.hip.model_stream(0)), lambda: b.context(b.hip.model_stream(0), batch=2),
                 lambda: b.context(b.hip.model_stream(0), hidden=64)):
        ctx = make()
        assert put(ctx, lanes_per_sample=0) < 0
        b.ok(put(ctx))
        b.L.mppi_destroy(ctx)


def case_autotune(b):
    """A context created with the library's choice can be tuned; the result names
    its shapes."""
    ctx = b.bicycle(2000, 60, "circles")
    report = C.create_string_buffer(1 << 16)
    b.ok(b.L.mppi_autotune(ctx, 1, report, len(report)))
    t = b.abi.Tuning()
    b.ok(b.L.mppi_get_tuning(ctx, C.byref(t)))
    assert t.lanes_per_sample > 0 and b"form=2" in report.value and b"form=1" in report.value
    b.ok(b.L.mppi_rollout(ctx))


CASES = {n[5:]: f for n, f in list(globals().items()) if n.startswith("case_")}


@pytest.mark.parametrize("name", sorted(CASES))
def test_ordering(model, name):
    run_case(model, name)


if __name__ == "__main__":
    CASES[sys.argv[2]](Bench(sys.argv[1]))
