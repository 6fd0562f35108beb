"""Solves at the edges of what they accept: streams that end before the handle,
sizes at the limit of the fixed workspace, values that are not finite."""
import ctypes as C

import numpy as np
import pytest
import torch

from gpu_util import rel2, say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def test_graph_workspace_outlives_its_stream():
    """A graph solve on a stream that is destroyed before the handle is freed: the
    workspace (328 MB of basis vectors) goes back to the pool."""
    import paper_1806_11558_amd as hm
    from paper_1806_11558_amd import _binding
    from synthetic import icosphere, normal_columns
    V, T = icosphere(4)
    f = torch.tensor(normal_columns(len(T), 8, seed=3), device=DEV)
    L = _binding.lib()                                  # the HIP runtime it is linked to
    say("graph workspace and its stream")
    for _ in range(2):                                  # second time: everything is loaded
        torch.cuda.synchronize()
        hm.release_memory()
        before = torch.cuda.mem_get_info()[0]
        st = C.c_void_p()
        assert L.hipStreamCreate(C.byref(st)) == 0
        H = hm.HMatrix(V, T, leaf_size=32, eps=1e-6, precision="f64")
        _, info, status = H.solve(f, tol=1e-6, restart=1000, graph=True, stream=st.value)
        assert status == hm.HM_OK
        assert L.hipStreamDestroy(st) == 0
        H.free()
        hm.release_memory()
        after = torch.cuda.mem_get_info()[0]
    assert before - after < 64 << 20, (before, after)
