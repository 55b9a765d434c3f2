"""Products with one operand of whole aligned chunks of 8 and one that is not, either way round.

Each operand takes its own path into LDS: 16-byte loads throughout where every row is whole aligned chunks,
else chunk by chunk (whole aligned chunks at once, the rest entry by entry).  Extents and strides here make
rows that are whole but not aligned, aligned but ragged at the end, and neither.  Tolerance: products of bf16
values summed in fp32, 5e-5 of the sum of the terms' magnitudes; a network with bf16 activations as the other
network cases.
"""

import numpy as np
import pytest
import torch

from test_gpu_surrogate import bf16_round, make
from test_gpu_surrogate_shapes import test_network_matches_oracle as network_matches_oracle

pytestmark = pytest.mark.gpu


def operand(x, along_k, stride, offset):
    """x (rows, k) in device memory, contiguous along k or along rows at the given stride, `offset` entries in."""
    y = x if along_k else x.T
    buf = torch.zeros(offset + y.shape[0] * stride, dtype=torch.bfloat16, device="cuda")
    view = buf[offset:].view(y.shape[0], stride)[:, :y.shape[1]]
    view.copy_(torch.as_tensor(y))
    return buf[offset:], ((stride, 1) if along_k else (1, stride))


@pytest.mark.parametrize("splits", [1, 2])  # every K here has two whole 32-deep splits
@pytest.mark.parametrize("ak", [True, False])
@pytest.mark.parametrize("bk", [True, False])
# (padding of the row stride, offset) of each operand: (0, 0) with extents that are multiples of 8 is whole and aligned
@pytest.mark.parametrize("M,N,K,a,b", [(64, 21, 136, (0, 0), (0, 0)), (72, 40, 264, (0, 0), (4, 0)), (72, 40, 264, (8, 0), (0, 1)),
                                       (21, 64, 136, (0, 0), (0, 0)), (40, 72, 264, (4, 0), (0, 0)), (40, 72, 264, (0, 1), (8, 0)),
                                       (30, 90, 100, (2, 0), (6, 0)), (12, 28, 324, (4, 4), (4, 4))])
def test_each_operand_takes_its_own_path(M, N, K, a, b, ak, bk, splits):
    h, _ = make()
    rng = np.random.default_rng(M + N + K)
    A, B = (rng.standard_normal(s).astype(np.float32) for s in ((M, K), (N, K)))
    dA, sa = operand(A, ak, (K if ak else M) + a[0], a[1])
    dB, sb = operand(B, bk, (K if bk else N) + b[0], b[1])
    C = h.debug_gemm(M, N, K, dA, *sa, dB, *sb, splits).sum(dim=0).cpu().numpy().astype(np.float64)
    Ar, Br = bf16_round(A), bf16_round(B)
    assert np.all(np.abs(C - Ar @ Br.T) <= 5e-5 * (np.abs(Ar) @ np.abs(Br).T) + 1e-30)


@pytest.mark.parametrize("channels", [(1, 12, 28, 52, 100), (1, 33, 65, 17, 9), (1, 32, 60, 24, 20)])
def test_networks_with_ragged_channels(channels):
    network_matches_oracle(16, 3, channels)
