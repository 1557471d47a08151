import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


@pytest.fixture(scope="session")
def oracle():
    import oracle as o
    o.lib()
    return o


@pytest.fixture(scope="session")
def kernels_of():
    """kernels_of(run): the (mangled) names of the kernels that run() launches on torch's current stream, found by recording
    the call into a graph that is never launched.  For tests of one form of a launch: that the rule still chooses it."""
    import ctypes
    import re
    import tempfile

    import torch

    def names(run):
        graph = torch.cuda.CUDAGraph(keep_graph=True)
        with torch.cuda.graph(graph):
            run()
        with open("/proc/self/maps") as f:
            loaded = sorted({line.split()[-1] for line in f if "libamdhip64" in line})
        hip = ctypes.CDLL(loaded[0])
        with tempfile.TemporaryDirectory() as d:
            dot = os.path.join(d, "graph.dot")
            rc = hip.hipGraphDebugDotPrint(ctypes.c_void_p(graph.raw_cuda_graph()), dot.encode(), ctypes.c_uint(1))
            assert rc == 0, f"hipGraphDebugDotPrint: {rc}"
            with open(dot) as f:
                return re.findall(r"_Z\w+", f.read())

    return names
