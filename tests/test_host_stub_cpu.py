"""The solver's host code on stand-ins for the HIP runtime and the launchers
(host_stub.cpp): failures of launches, which no test may provoke on a GPU, what
the kernel statistics count, and the order of streams."""
import ctypes as C
import os
import shutil
import subprocess

import pytest

import swf_workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def S():
    from paper_2512_16889_amd import swf
    return swf


@pytest.fixture(scope="module")
def lib(S, tmp_path_factory):
    if not shutil.which(HIPCC):
        pytest.skip("no hipcc")
    out = str(tmp_path_factory.mktemp("stub") / "libswf_stub.so")
    csrc = os.path.join(ROOT, "paper_2512_16889_amd", "csrc")
    objs = []
    for src in (os.path.join(csrc, "swf_api.cpp"), os.path.join(ROOT, "tests", "host_stub.cpp")):
        objs.append(out + os.path.basename(src) + ".o")
        subprocess.run([HIPCC, "-x", "hip", "--cuda-host-only", "--offload-arch=gfx950", "-O1", "-std=c++17", "-fPIC",
                        "-I", os.path.join(ROOT, "include"), "-I", csrc, "-c", src, "-o", objs[-1]], check=True)
    # there is no device code behind the host objects; their own symbols come first (the process may hold the
    # real runtime)
    names = subprocess.run(["nm", "-u"] + objs, check=True, capture_output=True, text=True).stdout.split()
    subprocess.run(["g++", "-shared", "-o", out] + objs + ["-Wl,-Bsymbolic"] +
                   [f"-Wl,--defsym={n}=0" for n in set(names) if n.startswith("__hip_fatbin")], check=True)
    lib = C.CDLL(out)
    lib.swf_last_error.restype = C.c_char_p
    lib.swf_last_error.argtypes = [C.c_void_p]
    lib.stub_fail.argtypes = [C.c_char_p, C.c_int]
    lib.stub_count.argtypes = [C.c_char_p]
    lib.stub_log.restype = C.c_char_p
    return lib


class Context:
    def __init__(self, S, lib, prob, **kw):
        grids, terms, ffirst, solves, verts, win = S.marshal(prob)
        opt = S.Options()
        opt.batched = 1
        for k, v in kw.items():
            setattr(opt, k, v)
        self.lib, self.ctx = lib, C.c_void_p()
        assert lib.swf_init(grids, len(prob.grids), terms, ffirst, len(prob.fields), solves, len(prob.solves), verts,
                            len(prob.vertices), C.byref(win), C.byref(opt), C.byref(self.ctx)) == 0, lib.swf_last_error(None)

    def __getattr__(self, name):
        return lambda *a: getattr(self.lib, "swf_" + name)(self.ctx, *a)

    def __enter__(self):
        return self

    def __exit__(self, *e):
        self.lib.swf_free(self.ctx)


@pytest.mark.parametrize("failing,at", [("finite_check", 1), ("stage_consts", 3), ("pass", 17)])
@pytest.mark.parametrize("restart", ["reset", "set_psi", "go on"])
def test_counter_after_a_failed_launch(S, lib, failing, at, restart):
    """Two of four steps are enqueued when a launch fails (the check after step 2, or one of step 3: 8 passes
    a step).  The device counter then stands at those two, and the next call starts where it says: a reset at
    0, a restored state at its index."""
    prob = W.config_2d(n=64, L=160.0, n_solves=1, steps=10)
    with Context(S, lib, prob, check_every=2) as c:
        assert c.step(1, None) == 0 and lib.stub_step() == 1
        assert c.reset() == 0 and lib.stub_step() == 0
        lib.stub_fail(failing.encode(), at)
        assert c.step(4, None) == S.SWF_E_HIP
        assert b"stub error" in c.last_error()
        assert lib.stub_step() == 2
        start = 2
        if restart == "reset":
            assert c.reset() == 0
            start = 0
        elif restart == "set_psi":
            psi = (C.c_double * (8 * 64 * 64))()
            assert c.set_psi(0, psi, 5) == 0
            start = 5
        assert c.step(1, None) == 0
        assert lib.stub_step_add() == 0 and lib.stub_step() == start + 1


@pytest.mark.parametrize("scheme", ["rk4", "dp5", "iprk4"])
@pytest.mark.parametrize("vertices", [0, 1])
def test_every_launch_of_a_step_is_timed(S, lib, scheme, vertices):
    """Of a step's kernels the statistics leave out the accumulation of the vertices alone.  Each interaction-picture
    pass moves the state arrays it reads and writes: Y -> YS; YS, Y -> YS, ACC; YS, ACC -> Y, the middle one in two
    halves (4 and 5 arrays) around the vertices' sums; four free evolutions of 6 (2D) or 2 (1D) passes' arrays."""
    prob = W.config_bw_1d(n=64, L=100.0, steps=4) if vertices else W.config_2d(n=64, L=160.0, n_solves=2, steps=10)
    w = prob.window
    prob.window = W.Window(w.t_in, w.t_out, w.dt, scheme)
    with Context(S, lib, prob, profile=1, stepper={"rk4": S.SWF_RK4, "dp5": S.SWF_DP5, "iprk4": S.SWF_IPRK4}[scheme]) as c:
        lib.stub_clear()
        assert c.step(3, None) == 0
        n, ms, by = C.c_longlong(), C.c_double(), C.c_double()
        launches, moved = 0, 0.0
        for kind in range(6):
            assert c.kernel_stats(kind, C.byref(n), C.byref(ms), C.byref(by)) == 0
            launches += n.value
            assert ms.value == n.value             # the stand-in's events are 1 ms apart
            if kind != 3:
                moved += by.value
        enqueued = sum(lib.stub_count(k.encode()) for k in ("pass", "stage_consts", "ip_point", "bw_stage"))
        assert lib.stub_count(b"stage_consts") == 3
        assert launches == enqueued
        if scheme == "iprk4":
            array = 4 * 16 * (64 if vertices else 64 * 64) * 2          # of both solves, in double
            points = 2 + (4 + 5 if vertices else 4) + 3
            assert moved == 3 * array * (points + 4 * (4 if vertices else 6))


def test_init_waits_for_the_callers_stream(S, lib):
    """The workspace is the caller's memory: what the caller has queued on it comes before the first upload.  A
    stream that is being captured has nothing to wait for, and is left alone."""
    prob = W.config_2d(n=64, L=160.0, n_solves=1, steps=10)
    for capturing in (0, 1):
        lib.stub_clear_log()
        lib.stub_capturing(capturing)
        with Context(S, lib, prob):
            calls = lib.stub_log().decode().splitlines()
        lib.stub_capturing(0)
        before = calls[:calls.index("write own")]
        assert before == ([] if capturing else ["record caller", "wait own"])
        assert "record caller" not in calls[len(before):] and "write caller" not in calls
