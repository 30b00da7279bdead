"""GPU kernels at the sizes where their tiling and dispatch change, against the oracle."""
import numpy as np
import pytest
import torch

import paper_1307_2666_amd as hif
from oracle.idqr import interp_decomp

from test_gpu_parity import _check_id

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n", [(40, 31), (256, 32), (257, 33), (511, 96), (4096, 64), (4097, 65), (4353, 129),
                                 (8200, 95), (32768, 48)])
def test_row_compression_tree_edges(m, n):
    # Row compression of problems at the edges of its tree: one chunk of at
    # most 256 rows, one group of at most 16 chunks, several groups; last
    # panels of fewer than 32 columns; three unequal problems in one batch.
    # The column scales make the pivots unique, so that the ID of R0 has the
    # oracle's skeleton and T.
    rng = np.random.default_rng(m + n)
    cases = []
    for mm, nn in ((m, n), (max(n + 1, m - 37), n), (m // 2 + n, max(2, n - 5))):
        cases.append(rng.standard_normal((mm, nn)) * (10.0 ** (-9.0 * np.arange(nn) / nn))[rng.permutation(nn)])
    tol = 1e-6
    out = hif.id_batched([torch.tensor(Y) for Y in cases], [tol] * len(cases))
    for Y, (sk, rd, T) in zip(cases, out):
        osk, _, oT = interp_decomp(Y, tol)
        _check_id(Y, tol, True, sk.numpy(), rd.numpy(), T.numpy(), osk, oT)
