"""Runs a test's body in a child process whose libsic is bound to the
recording runtime (recording_runtime.cpp) instead of the HIP runtime."""
import ctypes
import functools
import os
import subprocess
import sys
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.join(ROOT, "tests")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

rec = None  # the recording runtime, in the child


_folder = tempfile.TemporaryDirectory(prefix="sic_rec_")  # removed when the tests end


@functools.lru_cache(maxsize=None)
def _runtime() -> str:
    out = os.path.join(_folder.name, "librec.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-w", "-D__HIP_PLATFORM_AMD__",
                    "-I", os.path.join(ROCM, "include"), "-I", os.path.join(ROOT, "paper_1506_07207_amd", "csrc"),
                    "-o", out, os.path.join(HERE, "recording_runtime.cpp")], check=True)
    return out


def start(path: str):
    """In the child: the recording runtime's symbols first, then libsic."""
    global rec
    sys.modules["torch"] = None  # it would bring a HIP runtime of its own
    rec = ctypes.CDLL(path, mode=ctypes.RTLD_GLOBAL)
    rec.rec_launches.restype = rec.rec_events.restype = ctypes.c_char_p
    rec.rec_live.restype = ctypes.c_long
    rec.rec_fail_alloc.argtypes = [ctypes.c_long]
    rec.rec_fail_launch.argtypes = [ctypes.c_char_p, ctypes.c_long]
    from paper_1506_07207_amd import binding as B

    B.load()


def launches():
    """(kernel, grid, block, dynamic LDS bytes) of every launch since rec_clear."""
    rows = [line.rsplit(" ", 3) for line in rec.rec_launches().decode().splitlines()]
    return [(k, int(g), int(b), int(lds)) for k, g, b, lds in rows]


def events():
    return rec.rec_events().decode().splitlines()


def in_child(fn):
    @functools.wraps(fn)
    def run(**kw):
        from paper_1506_07207_amd import binding as B
        from paper_1506_07207_amd import build as hb

        if not os.path.exists(B.LIB_PATH):
            hb.build()
        code = (f"import sys; sys.path.insert(0, {ROOT!r})\n"
                f"from tests import host_runtime as H\nH.start({_runtime()!r})\n"
                f"import tests.{fn.__module__.split('.')[-1]} as m\nm.{fn.__name__}.__wrapped__(**{kw!r})\n")
        r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, r.stdout + r.stderr

    return run
