"""What the library's host code asks the HIP runtime for, without a GPU: calls run in a child process on a
stand-in runtime (fake_hip.c) that logs every allocation, device selection and launch with the device
that was current."""
import json
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes, json, os, sys
sys.path.insert(0, %r)
del os.environ["LD_PRELOAD"]
import numpy as np
from paper_2007_09884_amd import opmm
fake = ctypes.CDLL(None)
fake.fake_log.restype = ctypes.c_char_p
lib, P = opmm.lib, ctypes.c_void_p(1 << 20)       # P: a device pointer nobody reads

def lines():
    return [l.split(None, 5) for l in fake.fake_log().decode().splitlines()]

def records(S, T=57, n_cand=None):
    return opmm.saccade_records(np.full(S, T) if np.isscalar(T) else T, 2, np.full(S, 10.0), np.zeros(S),
                                np.full(S, 43.0), np.arange(S), n_cand)

def ptr(a):
    return a.ctypes.data_as(ctypes.c_void_p)

def check(rc):
    assert rc == 0, (rc, lib.opmm_last_error(ctx._h))

def fit_nm(recs, **kw):
    check(lib.opmm_fit_nm(ctx._h, P, 1 << 40, ptr(recs), len(recs), ctypes.byref(opmm.nm_params(**kw)), None, P, P,
                          None, None, None, None))

def polish(recs, **kw):
    check(lib.opmm_polish(ctx._h, P, 1 << 40, ptr(recs), len(recs), ctypes.byref(opmm.polish_params(**kw)), 18, P, P,
                          None, None, None, None))

def sensitivity(recs):
    check(lib.opmm_sensitivity(ctx._h, ptr(recs), len(recs), P, ctypes.c_float(1.0), P, P, None))

def ivt(N, max_out, min_dur=6.0):
    recs, n = np.zeros(max_out, opmm.SACCADE_DTYPE), ctypes.c_int32()
    check(lib.opmm_ivt_extract(ctx._h, P, N, ctypes.c_float(1.0), ctypes.c_float(30.0), ctypes.c_float(min_dur),
                               ctypes.c_float(0.0), 2048, ctypes.c_uint64(0), max_out, ptr(recs), P, 1 << 40, None,
                               ctypes.byref(n), None))

def fit(recs, **kw):
    check(lib.opmm_fit(ctx._h, P, 1 << 40, ptr(recs), len(recs), ctypes.byref(opmm.fit_params(**kw)), None, P, P,
                       None, None, None, None))

ctx = opmm.Context(0)
fake.fake_clear()
""" % ROOT


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    if os.environ.get("LD_PRELOAD"):
        pytest.skip("a preload is already set")
    include = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")
    so = str(tmp_path_factory.mktemp("fake") / "libfake_hip.so")
    subprocess.run(["gcc", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I" + include,
                    os.path.join(HERE, "fake_hip.c"), "-o", so], check=True)

    def run(code):
        r = subprocess.run([sys.executable, "-c", PRELUDE + code], cwd=ROOT, env=dict(os.environ, LD_PRELOAD=so),
                           capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stdout + r.stderr[-3000:]
        return json.loads(r.stdout.splitlines()[-1])
    return run


@pytest.mark.parametrize("call", ["ivt(100000, 4096)", "fit_nm(records(5))", "polish(records(5))",
                                  "sensitivity(records(5))", "fit(records(5))"])
def test_work_goes_to_the_contexts_device(fake, call):
    """Another device is current when the call comes: what it allocates and launches is on the context's."""
    log = fake("fake.fake_current(1)\n%s\nprint(json.dumps(lines()))" % call)
    work = [l for l in log if l[0] in ("malloc", "async", "launch")]
    assert any(l[0] == "launch" for l in work) and all(l[1] == "0" for l in work), work


@pytest.mark.parametrize("polish_iter", [0, 4])
def test_server_slots_fit_their_budget(fake, polish_iter):
    """Every per-slot array of a server counts against hbm_budget_bytes."""
    budget = 1000000
    log = fake("""
prm = opmm.serve_params(max_slots=1 << 20, max_T=1, hbm_budget_bytes=%d, polish_iter=%d)
sv = ctypes.c_void_p()
check(lib.opmm_server_create(ctx._h, None, ctypes.byref(prm), ctypes.byref(sv)))
print(json.dumps([lib.opmm_server_slots(sv), lines()]))""" % (budget, polish_iter))
    slots, log = log
    sizes = [int(l[2]) for l in log if l[0] == "malloc"]
    staged = 2 * 4 * min(slots, 4096)      # traces admitted in one step: the server's, not a slot's
    assert staged in sizes
    used = sum(sizes) - staged
    assert budget - used // slots < used <= budget


@pytest.mark.parametrize("N,max_out", [(100000, 4096), (200000000, 20000000)])
def test_extraction_allocates_for_what_it_finds(fake, N, max_out):
    """A stream without saccades costs no memory for records, however many the caller would take."""
    log = fake("ivt(%d, %d)\nprint(json.dumps(lines()))" % (N, max_out))
    assert sum(int(l[2]) for l in log if l[0] in ("malloc", "async", "pinned")) <= 1 << 20


ANCHORED = """
def anchored(recs, **kw):
    fake.fake_clear()
    fit(recs, n_rounds=10, screen_rounds=8, **kw)
    names = ["anchor" if "anchor" in l[5] else "verify" for l in lines()
             if l[0] == "launch" and ("anchor" in l[5] or "fit_verify" in l[5])]
    rounds = "".join("a" if n == "anchor" else "v" for n in names).replace("av", "A")
    assert len(rounds) == 8
    return [r for r, c in enumerate(rounds) if c == "A"]
"""


def test_anchor_where_it_pays(fake):
    """The rounds whose verify threshold comes from an anchor launch: those where it was measured to spare
    more than it costs, by the candidates' work, the width and the tolerance; not by how the tiles pad."""
    r = fake(ANCHORED + """
big, few = records(256), records(2000)
print(json.dumps(dict(
    default=anchored(big, n_cand=65536), wide=anchored(big, n_cand=65536, screen_tol=5e-3),
    tight=anchored(big, n_cand=65536, screen_tol=5e-6), one=anchored(records(1), n_cand=65536),
    padded=[anchored(few, n_cand=513, tile=t) for t in (1, 7)])))""")
    assert r["default"] in ([4, 5, 6, 7], [5, 6, 7])      # even at w = 1.6 %
    assert r["wide"] == [1, 2, 3, 4, 5, 6, 7]
    assert r["tight"] == [6, 7] or r["tight"] == [5, 6, 7]
    assert r["one"] == []
    assert r["padded"] == [[], []]


def test_simplex_tasks_per_wave(fake):
    """Saccades per wave of the simplex search (batch over grid): one while every task has a SIMD of its own or shares
    it with a much shorter one, three where it shares it with one of like length, and beyond two per SIMD."""
    r = fake("""
def grid(T):
    fake.fake_clear()
    fit_nm(records(len(T), np.asarray(T)))
    return [int(l[2]) for l in lines() if l[0] == "launch" and "nm_kernel" in l[5]]

spread = lambda S: np.linspace(20, 150, S).astype(int)
print(json.dumps([grid(np.full(1024, 57)), grid(np.full(1025, 57)), grid(spread(1025)), grid(spread(1500)),
                  grid(spread(1900)), grid(spread(2049)), grid(np.full(1500, 1025)), grid([2048] + [20] * 1500)]))""")
    assert r == [[1024], [342], [1025], [1500], [634], [683], [1500], [1501]]


def test_autotuner_times_each_kernel_once(fake):
    """Shapes that run the same kernel are one candidate; the pick is the lowest index of its kernel."""
    launches, pick, small = fake("""
recs, prm, t = records(64), opmm.fit_params(n_cand=65536, n_rounds=2), ctypes.c_int32(-1)
check(lib.opmm_autotune(ctx._h, P, 1 << 40, ptr(recs), len(recs), ctypes.byref(prm), ctypes.byref(t), None))
tuned = lines()
c2 = opmm.Context(0)
small = []
for n in (1 << 20, 2048, 2047, 1024, 1023, 512, 511, 1):     # the library's own choice, by candidates
    fake.fake_clear()
    r = records(3000)
    assert lib.opmm_fit(c2._h, P, 1 << 40, ptr(r), 3000, ctypes.byref(opmm.fit_params(n_cand=n)), None, P, P, None, None,
                        None, None) == 0
    small += [l[5].split("fit_round_kernel")[1][:11] for l in lines() if l[0] == "launch" and "fit_round" in l[5]]
print(json.dumps([tuned, t.value, small]))""")
    kernels = [l[5] for l in launches if l[0] == "launch" and "fit_round" in l[5]]
    assert len(set(kernels)) == 7 and all(kernels.count(k) == 2 * 3 for k in set(kernels))
    assert pick == 0
    assert small == ["ILi256ELi8E"] * 2 + ["ILi256ELi4E"] * 2 + ["ILi256ELi2E"] * 4
