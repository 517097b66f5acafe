"""When the read slots and their helper threads exist, and that they disturb
nothing: each case in a process of its own, which counts its threads and holds
no other handles."""
import os
import subprocess
import sys
import textwrap

import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PRELUDE = """
import ctypes as C, os, sys, threading
import numpy as np, torch
from paper_1711_02003_amd import lbcg as L, workloads as W
assert torch.cuda.is_available()
helpers = min(7, len(os.sched_getaffinity(0)) - 1)

def threads():
    return len(os.listdir("/proc/self/task"))

def lattice(dims):
    rng = np.random.default_rng(1)
    rR, rB = W.colour_densities(rng.uniform(-0.9, 0.9, dims[::-1]))
    return L.Sim("D3Q19", dims, 1.2, 0.7, 0.01, 0.7).init_fields(rR, rB).step(2)

def read(s, out):
    p = [C.cast(a, C.POINTER(C.c_double)) for a in out]
    assert L.load_library().lbcg_fields(s._handle(), *p) == 0

s = lattice((20, 20, 20))
s.fields()
s.close()
base = threads()
"""


def _run(code):
    if not __import__("torch").cuda.is_available():
        pytest.skip("no GPU")
    env = dict(os.environ, PYTHONPATH=ROOT, OMP_NUM_THREADS="1")
    r = subprocess.run([sys.executable, "-u", "-c", PRELUDE + textwrap.dedent(code)], cwd=ROOT, env=env,
                       capture_output=True, text=True, timeout=100)
    print(r.stdout[-2000:], flush=True)
    assert r.returncode == 0, r.stderr[-3000:]


def test_one_lattice_at_a_time_reads_without_slots():
    # 4.4 MB a read: a program that reads each lattice once does not pay for
    # slots and threads; one that goes on reading gets them with the third read
    _run("""
        for _ in range(3):
            s = lattice((45, 38, 53))
            f = s.fields()
            assert threads() == base, (threads(), base)
            s.close()
        s = lattice((45, 38, 53))
        n = []
        for _ in range(4):
            g = s.fields()
            n.append(threads() - base)
            assert all(np.array_equal(f[k], g[k]) for k in f)
        assert n == [0, 0, helpers, helpers], n
        s.close()
        assert threads() == base
        # a large read pays for them at once
        s = lattice((96, 96, 96))
        s.fields()
        assert threads() == base + helpers
        s.close()
        assert threads() == base
    """)


def test_pinned_destinations_are_written_by_the_device():
    # no slots, no helpers; sizes around a slot's chunk of nodes, then the same
    # reads into pageable memory, with and without slots
    _run("""
        for dims in ((61, 47, 43), (56, 56, 56), (83, 81, 79)):
            s = lattice(dims)
            n = s.N
            pin = [torch.full((k * n,), float("nan"), dtype=torch.float64, pin_memory=True) for k in (1, 1, 3, 1)]
            base = threads()  # torch has threads of its own for these
            for _ in range(4):
                read(s, [t.data_ptr() for t in pin])
                assert threads() == base, (threads(), base)
            for _ in range(4):
                f = s.fields()
                for k, t in zip(("rhoR", "rhoB", "u", "psi"), pin):
                    assert np.array_equal(f[k].ravel(), t.numpy())
            assert threads() == base + helpers
            s.close()
    """)


def test_last_handle_goes_during_a_capture_of_another_thread():
    # the slots are given back while this thread captures in global mode; the
    # handle lives in memory and on a stream of the caller's, so that nothing
    # else is freed with it
    _run("""
        side = torch.cuda.Stream()
        x = torch.zeros(1000, device="cuda")
        y = torch.empty_like(x)
        for use in (1, 2):
            rng = np.random.default_rng(1)
            rR, rB = W.colour_densities(rng.uniform(-0.9, 0.9, (80, 80, 80)))
            s = L.Sim("D3Q19", (80, 80, 80), 1.2, 0.7, 0.01, 0.7, stream=side.cuda_stream).init_fields(rR, rB).step(2)
            f = s.fields()
            assert threads() >= base + helpers
            keep = s._buf
            torch.cuda.synchronize()
            done = []
            def gone():
                s.close()
                done.append(threads())
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, capture_error_mode="global"):
                y.copy_(x + 1)
                t = threading.Thread(target=gone)
                t.start()
                t.join()
                x.copy_(y)
            assert len(done) == 1
            for k in range(3):
                x.fill_(10 * use + k)
                g.replay()
                torch.cuda.synchronize()
                assert float(x[7]) == 10 * use + k + 1
            del g, keep
    """)


def test_read_with_another_device_current():
    import torch
    if torch.cuda.device_count() < 2:
        pytest.skip("needs two GPUs: a read of a handle on the second while the first is current")
    _run("""
        with torch.cuda.device(1):
            s = lattice((96, 96, 96))
            want = s.fields()
        for _ in range(2):
            got = s.fields()  # device 0 is current
            assert all(np.array_equal(got[k], want[k]) for k in want)
        s.close()
    """)


def test_overlapping_destinations_hold_the_last_row():
    # one place for several rows: it holds the last of them, as with plain copies
    _run("""
        s = lattice((96, 96, 96))
        n = s.N
        f = [s.fields() for _ in range(2)][1]  # the slots exist
        buf = np.empty(3 * n)
        for _ in range(30):
            buf[:] = np.nan
            read(s, [buf[:n].ctypes.data, None, None, buf[:n].ctypes.data])
            assert np.array_equal(buf[:n], f["psi"].ravel())
            read(s, [buf[:n].ctypes.data, buf[n:2 * n].ctypes.data, buf.ctypes.data, buf[2 * n:].ctypes.data])
            assert np.array_equal(buf[:2 * n], f["u"].reshape(-1)[:2 * n])
            assert np.array_equal(buf[2 * n:], f["psi"].ravel())
    """)
