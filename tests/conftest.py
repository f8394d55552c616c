import ctypes
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
    from oracle import build as obuild
    obuild.build()
    from oracle import agq_oracle
    return agq_oracle


@pytest.fixture(scope="session")
def gemm_route():
    """route(M, K, Ns, ...): the kernel that the library's dispatch picks for a linear layer, by the same host code (the
    probe library is compiled from the library's own header): "stream" (weight-streaming kernel) or a variant of the tiled
    kernel, "128", "split", "64" or "64x2".  A test of a variant asserts it, so that a change of the dispatch rules cannot
    take the test off its path unseen."""
    from paper_2312_05693_amd import build
    if not os.path.exists(build.PROBE_LIB):
        build.build()
    probe = ctypes.CDLL(build.PROBE_LIB)
    names = {-1: "stream", 0: "128", 1: "split", 2: "64", 3: "64x2"}

    def route(M, K, Ns, x_kind=0, n_extra=-1, workspace_bytes=1 << 40):
        return names[probe.agq_probe_gemm_route(x_kind, ctypes.c_int64(M), ctypes.c_int64(K), (ctypes.c_int64 * len(Ns))(*Ns),
                                                len(Ns), n_extra, ctypes.c_size_t(workspace_bytes))]
    return route
