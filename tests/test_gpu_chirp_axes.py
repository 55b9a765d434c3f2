"""The chirp-z transform on every axis of every pass that can run it.

Each case names the transform its axes take, so that a change of the rule that moves a length elsewhere
fails here and does not empty the test.  Lengths: primes above the limits of the direct stages, short
enough that the buffers of all components fit.  Bounds are those of the same
checks on other axes: 1e-13 for one projection, operator or transform, 1e-10 (fields) and 1e-11
(homogenized) for solves; at a CG tolerance of 1e-11 the passes are those of the CG on displacements, at
1e-12 those of the CG on strain fields.
"""

import numpy as np
import pytest

from helpers import field_err, lame_fields, ncomp, pack, rel
from oracle import materials, spectral
from paper_2408_03804_amd import binding, workloads
from test_gpu_solver import TOL_FIELD, TOL_HOMOG, make, run_both
from test_gpu_stages import random_state

pytestmark = pytest.mark.gpu

D, C = "direct", "chirp"
# shape (z, y, x) or (y, x), strain, transforms of the axes
CASES = [((4, 433, 6), "small", (D, C, D)), ((4, 433, 6), "finite", (D, C, D)),
         ((283, 5, 4), "small", (C, D, D)), ((307, 4, 5), "finite", (C, D, D)), ((433, 3, 4), "finite", (C, D, D)),
         ((3, 4, 433), "small", (D, D, C)),
         ((4, 311, 6), "finite", (D, C, D)), ((3, 2, 379), "finite", (D, D, C)), ((4, 379, 3), "small", (D, C, D)), ((5, 379), "small", (D, C)),
         ((6, 433), "small", (D, C)), ((433, 6), "finite", (C, D)), ((5, 439), "finite", (D, C)), ((283, 433), "small", (C, C))]
IDS = ["%s-%s" % ("x".join(map(str, s)), k) for s, k, _ in CASES]


def law(kin):
    return "linear_elastic" if kin == "small" else "neo_hookean"


@pytest.fixture(autouse=True)
def the_axes_take_the_transform_the_case_is_for(request):
    c = request.node.callspec.params["case"]
    assert binding.fft_homog_debug_axis_plans(binding.make_desc(c[0], c[1], law(c[1]), 2)) == c[2]


def random_tensor(shape, kin, seed):
    A = np.random.default_rng(seed).standard_normal(tuple(shape) + (len(shape),) * 2)
    return 0.5 * (A + np.swapaxes(A, -1, -2)) if kin == "small" else A


@pytest.mark.parametrize("case", CASES, ids=IDS)
def test_transform_and_projection(case):
    import torch
    shape, kin, _ = case
    h = make(shape, kin, law(kin), tangent=True)
    x = np.random.default_rng(4).standard_normal((2, ncomp(kin, len(shape))) + shape)
    ref = np.fft.rfftn(x, axes=tuple(range(2, 2 + len(shape))))
    assert np.abs(h.debug_rfft(x).cpu().numpy() - ref).max() < 1e-13 * np.abs(ref).max()
    assert np.abs(h.debug_irfft(ref).cpu().numpy() - x).max() < 1e-13 * np.abs(x).max()
    A = random_tensor(shape, kin, 5)
    p = pack(A, kin == "small")
    out = h.debug_project(p[None]).cpu().numpy()[0]
    assert field_err(out, pack(spectral.apply_G(A, kin), kin == "small")) < 1e-13
    xin = torch.as_tensor(p[None]).cuda()
    na = torch.full_like(xin, float("nan"))
    binding.fft_homog_project_noalloc(binding.make_desc(shape, kin, law(kin), 2), xin, na)
    assert field_err(na.cpu().numpy()[0], out) < 1e-13


@pytest.mark.parametrize("k_mode", [0, 1])
@pytest.mark.parametrize("case", CASES, ids=IDS)
def test_operator(case, k_mode):
    shape, kin, _ = case
    d, small = len(shape), kin == "small"
    h = make(shape, kin, law(kin), k_mode=k_mode)
    phase = workloads.random_phases(shape, 2, 6)
    table = [[1.0, 1.0], [6.0, 3.0]]
    h.set_material(phase, table)
    E = random_state(shape, kin, 7, 0.05)
    h.set_field(np.moveaxis(E.reshape(tuple(shape) + (d * d,)), -1, 0), np.zeros(ncomp(kin, d)))
    p = random_tensor(shape, kin, 8)
    q = h.debug_apply_operator(pack(p, small)[None]).cpu().numpy()[0]
    lam, mu = lame_fields(phase, table)
    K = materials.MATERIALS[law(kin)].tangent_apply(E, p, lam, mu)
    assert field_err(q, pack(spectral.apply_G(K, kin), small)) < 1e-13


@pytest.mark.parametrize("tol_cg", [1e-11, 1e-12])
@pytest.mark.parametrize("case", CASES, ids=IDS)
def test_solve(case, tol_cg):
    shape, kin, _ = case
    d = len(shape)
    macro = np.r_[1e-2, np.zeros(2 if d == 2 else 5)] if kin == "small" else (np.eye(d) + 0.01 * np.arange(d * d).reshape(d, d) / 8).reshape(-1)
    o = run_both(shape, kin, law(kin), workloads.random_phases(shape, 2, 11), [[2.0, 1.0], [10.0, 5.0]], macro, 1, tol_cg=tol_cg)
    assert o["st"]["status"] == "ok" and abs(o["st"]["newton"] - o["ref"]["stats"]["newton"]) <= 1
    assert o["field_err"] < TOL_FIELD and o["stress_err"] < TOL_FIELD
    assert rel(o["S"], o["ref"]["macro_stress"]) < TOL_HOMOG
