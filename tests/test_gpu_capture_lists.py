"""A captured graph writes a tile list that is first used in it once, not again for
every step."""
import ctypes

import numpy as np
import pytest

from tests.gpu_common import DEV, dev, heff_operands, host, lib_heff, require_gpu, torch
from paper_2401_01921_amd import bst

pytestmark = pytest.mark.gpu


def _nodes(graph):
    hip = ctypes.CDLL("libamdhip64.so")
    n = ctypes.c_size_t()
    assert hip.hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    return n.value


def _capture(plan, ins, out, ws):
    g = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(g):
        plan.execute(ins, [out], ws)
    n = _nodes(g)
    g.instantiate()
    return g, n


def test_lists_are_written_once():
    require_gpu()
    specs, O = heff_operands(2, chi=96, qmax=4)
    plan = lib_heff(specs, "fp64")[1]
    ins = [dev(O[n].data) for n in ("L", "W1", "W2", "R", "psi")]
    ws = bst.workspace(plan.workspace_bytes)
    out = torch.empty(O["psi"].numel, dtype=torch.float64, device=DEV)
    plan.execute(ins, [out], ws)
    torch.cuda.synchronize()
    graphs = []
    for tile in (6, 7):   # both GEMM steps on a shape not used before, then on another
        plan.set_precision("fp32")
        plan.set_tile("fp32", tile)
        graphs.append(_capture(plan, ins, out, ws))
    plan.execute(ins, [out], ws)   # now the lists are there
    want = host(out)
    g, plain = _capture(plan, ins, out, ws)
    print("nodes", [n for _, n in graphs], "without lists", plain, flush=True)
    # two lists fit the arguments of one launch; the second graph writes all
    # four, the first one's too, which two launches hold
    first, second = (n - plain for _, n in graphs)
    assert first == 1 and second <= 2
    for graph in [g] + [x for x, _ in graphs]:
        for rep in range(3):
            out.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            assert torch.randn(1000, device=DEV).sum().isfinite().item()   # eager work between replays
            assert np.array_equal(host(out), want), rep
