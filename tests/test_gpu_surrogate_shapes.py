"""The surrogate's kernels at the sizes where their tiles and their dispatch change.

Tiles are 64 x 64 with 128-deep stages, loaded 16 bytes at a time where every row is whole aligned
chunks of 8 and entry by entry elsewhere; conv blocks gather their operands (input channels a multiple
of 8) and form their input gradient per parity class (output channels too), or expand them in memory.
Tolerances are those of the two roundings they test: products of bf16 values summed in fp32 to 5e-5 of
the sum of the terms' magnitudes, networks with bf16 activations and gradients to 2e-2 of the largest
output and 5e-2 (2-norm, each parameter block) of the gradient.
"""

import numpy as np
import pytest
import torch

from oracle import surrogate as OS
from test_gpu_surrogate import bf16_round, make, random_theta, rounded_weights

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ak", [True, False])
@pytest.mark.parametrize("bk", [True, False])
@pytest.mark.parametrize("M,N,K", [(64, 64, 128), (65, 72, 129), (8, 136, 120), (72, 8, 160), (1, 1, 1), (63, 21, 300)])
def test_gemm_at_tile_edges(M, N, K, ak, bk):
    h, _ = make()
    rng = np.random.default_rng(M + N + K)
    A, B = (rng.standard_normal(s).astype(np.float32) for s in ((M, K), (N, K)))
    dev = [torch.as_tensor(x if c else x.T.copy()).to(torch.bfloat16).cuda() for x, c in ((A, ak), (B, bk))]
    sa, sb = (K, 1) if ak else (1, M), (K, 1) if bk else (1, N)
    C = h.debug_gemm(M, N, K, dev[0], *sa, dev[1], *sb, 1)[0].cpu().numpy().astype(np.float64)
    Ar, Br = bf16_round(A), bf16_round(B)
    assert np.all(np.abs(C - Ar @ Br.T) <= 5e-5 * (np.abs(Ar) @ np.abs(Br).T) + 1e-30)


@pytest.mark.parametrize("n,batch,channels", [
    (16, 3, (1, 5, 8, 12, 6)),       # nothing in chunks of 8 but block 3's input
    (16, 5, (1, 8, 24, 40, 72)),     # channels that are no multiple of 32; one voxel left after block 4
    (16, 1, (1, 72, 136, 16, 8)),    # more than one column tile, stages that end inside a tap
    (48, 1, (1, 8, 16, 24, 32)),     # an odd edge (3) after block 4
    (16, 2, (1, 8, 20, 8, 16)),      # gathered operand, input gradient through memory
])
def test_network_matches_oracle(n, batch, channels):
    h, cfg = make(max_batch=batch, n=n, channels=channels)
    theta, kw = random_theta(cfg, 7)
    h.set_params(theta)
    rng = np.random.default_rng(8)
    phase = (rng.random((batch, n, n, n)) < 0.4).astype(np.uint8)
    feat = rng.standard_normal((batch, 1)).astype(np.float32)
    target = rng.standard_normal((batch, 21)).astype(np.float32)
    th = rounded_weights(theta, kw)
    ref = OS.predict(th, phase, bf16_round(feat), **kw)
    assert np.abs(h.forward(phase, feat).cpu().numpy() - ref).max() < 2e-2 * np.abs(ref).max()
    loss, g = h.loss_grad(phase, feat, target)
    Lr, gr = OS.loss_and_grad(th, phase, bf16_round(feat), target, **kw)
    assert abs(loss - Lr) < 2e-2 * abs(Lr)
    g = g.cpu().numpy()
    off = 0
    for name, shape in OS.param_shapes(**kw):
        m = int(np.prod(shape))
        assert np.linalg.norm(g[off:off + m] - gr[off:off + m]) < 5e-2 * np.linalg.norm(gr[off:off + m]) + 1e-12, name
        off += m
