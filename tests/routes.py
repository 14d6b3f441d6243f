"""What the planner decides, from a host build of its header: for tests that say which routine they reach."""
import functools
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
NONE, DEPTHWISE_3X3, SHORT_ROWS, SMALL, STEM, K9 = 0, 3, 4, 5, 8, 9   # families
SMALL_TENSOR = 16384   # weights below which a tensor of a rarer shape stays with the generic routine


@functools.lru_cache(maxsize=None)
def _program():
    exe = os.path.join(tempfile.mkdtemp(), "host_routes")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2202_07471_amd", "csrc"),
                           os.path.join(ROOT, "tests", "host_routes.cpp"), "-o", exe])
    return exe


def _ask(lines, *args):
    text = "".join(" ".join(str(int(x)) for x in line) + "\n" for line in lines)
    out = subprocess.run([_program(), *args], input=text, capture_output=True, text=True, check=True).stdout
    return [tuple(int(x) for x in line.split()) for line in out.splitlines()]


def routes(shapes, aligned=True):
    """(family, kernels a thread, threads) of each shape [cout, cin, kh, kw]."""
    return _ask([(m, n, kh * kw, aligned) for m, n, kh, kw in shapes])


def row_shapes(launches):
    """(vectors a thread, threads) of launches of 1x1 / FC rows with SQuant-C: (longest row, rows, bytes moved, binary32
    output) each."""
    return _ask(launches, "rows")


def enough(cin, elements, at_least=1):
    """Output channels with which a tensor is no small one."""
    return max(at_least, -(-SMALL_TENSOR // (cin * elements)))
