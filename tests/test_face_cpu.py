"""The Python face's native half where there is no GPU: exceptions out of the library."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

def run(code, *args):
    return subprocess.run([sys.executable, "-W", "always", "-c", code, *map(str, args)], cwd=ROOT, capture_output=True, text=True, timeout=300)


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
