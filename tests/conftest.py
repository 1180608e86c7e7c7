import ctypes
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu on the GPU box)")


def _gpu_available():
    try:
        import torch
        return torch.cuda.is_available()
    except Exception:
        return False


def pytest_collection_modifyitems(config, items):
    if _gpu_available():
        return
    skip = pytest.mark.skip(reason="no GPU in this process")
    for item in items:
        if "gpu" in item.keywords:
            item.add_marker(skip)


RULES_SOURCE = r"""
#include "gss_rules.h"
extern "C" void istft_plan(long S, long T, int num_cu, long* out) {
  const IstftPlan p = plan_istft(S, T, num_cu);
  out[0] = p.waves; out[1] = p.steps; out[2] = p.per_seg;
}
extern "C" int em_whole(int D, double load, int tiles, int ragged) { return use_whole(D, load, tiles, ragged != 0); }
extern "C" int em_quad(int D, int K, double load, int tiles, int iters, int lengths) { return use_quad(D, K, load, tiles, iters, lengths); }
"""


@pytest.fixture(scope="session")
def rules(tmp_path_factory):
    """The library's rules for choosing between kernels (csrc/gss_rules.h), built by the host compiler alone."""
    d = tmp_path_factory.mktemp("rules")
    (d / "rules.cpp").write_text(RULES_SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_2212_05271_amd", "csrc"),
                    str(d / "rules.cpp"), "-o", str(d / "rules.so")], check=True)
    lib = ctypes.CDLL(str(d / "rules.so"))

    class Rules:
        @staticmethod
        def istft(S, T, num_cu=256):
            """(wavefronts per workgroup, steps per workgroup, workgroups per segment) of gss_istft."""
            out = (ctypes.c_long * 3)()
            lib.istft_plan(ctypes.c_long(S), ctypes.c_long(T), ctypes.c_int(num_cu), out)
            return tuple(out)

        @staticmethod
        def em_one_launch(D, S, T, ragged=False, F=513, num_cu=256):
            """Whether gss_cacgmm_em takes the whole-EM kernel with one wavefront per problem (5 to 8 channels)."""
            return bool(lib.em_whole(D, ctypes.c_double(S * F / num_cu), (T + 63) // 64, int(ragged)))

        @staticmethod
        def em_four_wavefronts(D, K, S, T, iters, ragged=False, F=513, num_cu=256):
            """Whether gss_cacgmm_em takes four wavefronts per problem (where it runs a problem in one workgroup)."""
            return bool(lib.em_quad(D, K, ctypes.c_double(S * F / num_cu), (T + 63) // 64, iters, S if ragged else 1))

    return Rules
