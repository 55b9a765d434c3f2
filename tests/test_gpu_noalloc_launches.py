"""The allocation-free projection makes its tables on each call: one launch for all axes, whether they
run radix stages or the folded dense DFT (a chirp-z axis adds one).  Counted from a captured call; the
captured call replays to the eager call's bits.
"""

import ctypes

import numpy as np
import pytest

from helpers import field_err
from paper_2408_03804_amd import binding

pytestmark = pytest.mark.gpu


def graph_nodes(g):
    lib = binding.load_library()  # resolves the HIP runtime it is linked with
    n = ctypes.c_size_t(0)
    assert lib.hipGraphGetNodes(ctypes.c_void_p(g.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    return n.value


@pytest.mark.parametrize("shape,kin,mat,launches", [
    ((33, 36, 40), "small", "linear_elastic", 6), ((20, 18, 17), "finite", "neo_hookean", 6),
    ((33, 9, 8), "finite", "neo_hookean", 6), ((31, 50), "small", "linear_elastic", 4),
    ((8, 9, 10), "small", "linear_elastic", 6), ((4, 439, 6), "small", "linear_elastic", 7), ((283, 16), "small", "linear_elastic", 5)])
def test_one_table_launch(shape, kin, mat, launches):
    import torch
    d = binding.make_desc(shape, kin, mat, 2)
    c = {("small", 2): 3, ("small", 3): 6, ("finite", 3): 9}[kin, len(shape)]
    x = torch.as_tensor(np.random.default_rng(2).standard_normal((1, c) + shape)).cuda()
    out, ref = torch.empty_like(x), torch.empty_like(x)
    binding.fft_homog_project_noalloc(d, x, ref)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(g):
        binding.fft_homog_project_noalloc(d, x, out)
    assert graph_nodes(g) == launches
    g.instantiate()
    for _ in range(3):
        out.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref)
    h = binding.FFTHomog(shape, kin, mat, 2)
    # the handle's tables differ by their rounding only, as in the eager call's own test
    assert field_err(out.cpu().numpy(), h.debug_project(x).cpu().numpy().reshape(x.shape)) < 1e-13
