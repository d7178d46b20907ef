"""The Python face's native half where there is no GPU: arguments that it leaves to the Python functions, exceptions out of the
library, and a package without it or with one for another torch."""
import os
import shutil
import struct
import subprocess
import sys
import time

import numpy as np
import pytest

from paper_2409_15355_amd import binding as ba

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CALLS = {"encode_blocks": (10, 6), "reencode_positions": (10, 3), "final_block": (14, 8), "final_block_static": (13, 8),
         "final_block_cached": (18, 8), "prompts": (12, 7), "prompts_backward": (14, 10)}  # arguments, the first array


def run(code, *args):
    return subprocess.run([sys.executable, "-W", "always", "-c", code, *map(str, args)], cwd=ROOT, capture_output=True, text=True, timeout=300)


@pytest.mark.parametrize("call", CALLS)
@pytest.mark.parametrize("array", [[0, 100], np.array([0, 100]), np.array([0, 7, 100], dtype=np.int32)[::2], (0, 100)])
def test_lists_and_other_arrays_are_left_to_the_python_function_without_an_exception(call, array):
    """Looking at them costs a few calls of nothing, not the microseconds of a C++ exception (some forty of them)."""
    n_args, at = CALLS[call]
    take = getattr(ba._face(), call)
    heads = ba.Heads(8, 2, 64)
    args = [heads] + [None] * (at - 1) + [array] + [None] * (n_args - at - 1)
    assert take(*args) is None

    def once(*a):
        best = float("inf")
        for _ in range(20):
            t = time.perf_counter()
            for _ in range(200):
                take(*a)
            best = min(best, time.perf_counter() - t)
        return best

    assert once(*args) < 12 * once()  # (no arguments: refused at once)


def test_an_exception_inside_the_library_is_raised(tmp_path):
    """... with the interpreter's lock taken back, and not taken for an argument that the native half leaves alone."""
    src, lib = tmp_path / "throws.cpp", tmp_path / "throws.so"
    src.write_text('#include <new>\n#include <stdexcept>\nextern "C" int memory() { throw std::bad_alloc(); }\n'
                   'extern "C" int other() { throw std::runtime_error("x"); }\n')
    subprocess.run(["g++", "-shared", "-fPIC", "-o", str(lib), str(src)], check=True)
    r = run("""
import ctypes, sys
import numpy as np
from paper_2409_15355_amd import binding as ba
face, lib = ba._face(), ctypes.CDLL(sys.argv[1])
class Stream: cuda_stream = 0
offs = np.array([0, 4], dtype=np.int32)
for name, kind in (("memory", MemoryError), ("other", RuntimeError)):
    face.setup(ba.Heads, None, None, (ctypes.cast(getattr(lib, name), ctypes.c_void_p).value,) * 7)
    for _ in range(3):
        try:
            face.encode_blocks(ba.Heads(4, 4, 64), None, None, None, None, None, offs, 1, None, Stream())
            print("nothing raised")
        except kind:
            print("raised")
""", lib)
    assert r.returncode == 0 and r.stdout.split("\n")[:-1] == ["raised"] * 6, (r.returncode, r.stdout, r.stderr)


USE = """
import sys
sys.path.insert(0, sys.argv[1])
import numpy as np, torch
if len(sys.argv) > 2:
    torch.__version__ = sys.argv[2]
from paper_2409_15355_amd import binding as ba
heads, q = ba.Heads(4, 4, 64), torch.zeros((4, 4, 64), dtype=torch.bfloat16)
assert ba.ba_encode_blocks_workspace_bytes(heads, [0, 4]) > 0 and ba._face().prompts() is None
try:
    ba.ba_encode_blocks(heads, q, q, q, q, None, np.array([0, 4], dtype=np.int32))
except ValueError as e:
    print(type(ba._face()).__name__, "|", e)
"""


def test_the_native_half_has_no_thread_locals():
    """... which would slow down everybody else's, see build_face."""
    ba.load()
    with open(ba.FACE_PATH, "rb") as f:
        elf = f.read()
    at, = struct.unpack_from("<Q", elf, 32)
    size, n = struct.unpack_from("<HH", elf, 54)
    kinds = [struct.unpack_from("<I", elf, at + i * size)[0] for i in range(n)]
    assert 1 in kinds and 7 not in kinds  # PT_LOAD, PT_TLS


def test_the_package_works_without_its_native_half(tmp_path):
    pkg = tmp_path / "paper_2409_15355_amd"
    shutil.copytree(os.path.join(ROOT, "paper_2409_15355_amd"), pkg, ignore=shutil.ignore_patterns("_face.so", "_build", "csrc", "__pycache__"))
    r = run(USE, tmp_path)
    assert r.returncode == 0 and "_NoNative | q: expected a tensor in GPU memory" in r.stdout and "is missing" in r.stderr, (r.stdout, r.stderr)


def test_a_native_half_for_another_torch_is_left_alone():
    r = run(USE, ROOT, "1.2.3+x")
    assert r.returncode == 0 and "_NoNative | q: expected" in r.stdout and "this is 1.2.3+x" in r.stderr, (r.stdout, r.stderr)
    r = run(USE, ROOT)
    assert r.returncode == 0 and "module | q: expected" in r.stdout and "RuntimeWarning" not in r.stderr, (r.stdout, r.stderr)
