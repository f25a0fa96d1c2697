"""The team barriers of more kernels sit in uniform control flow (CPU only; see
test_barrier_uniformity): the initial search with 3-opt, 4-wave teams with long
candidate lists, and the batched kernel."""
import os

import pytest

from tests.test_barrier_uniformity import HIPCC, OPT, ROOT, _uniformity

pytestmark = pytest.mark.skipif(not (os.path.exists(HIPCC) and os.path.exists(OPT)),
                                reason="ROCm compiler not found")


@pytest.mark.parametrize("header,inst", [
    ("faco_init.hpp", "template __global__ void faco::init_search_kernel<16>(faco::Inst, int);"),
    ("faco_kernels.hpp", "template __global__ void faco::ant_kernel<32, 4>(faco::Inst, int);"),
    ("faco_kernels.hpp", "template __global__ void faco::ant_batch_kernel<32, 4>("
                         "const faco::Inst *, const int2 *, int, int, int);"),
])
def test_barriers_in_uniform_control_flow(tmp_path, header, inst):
    src = os.path.join(ROOT, "paper_2203_02228_amd", "csrc", header)
    st, bad = _uniformity(f'#include "{src}"\n{inst}\n', tmp_path)
    assert st["barriers"] >= 5, st
    assert bad == [], f"barriers under divergent branches: {bad[:4]}"
