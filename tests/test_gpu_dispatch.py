"""Each branch of the size-dependent dispatches at its edges, against the float64 oracle."""
import numpy as np
import pytest
import torch

import oracle as O
from gpu_util import DEV, note, rel_frob, to_np
from paper_2607_07964_amd import kronq as K

pytestmark = pytest.mark.gpu


# ---------------------------------------------------------------- fp32 covariance tile sizes
# 16-, 32- and 64-edge tiles (the largest that gives every CU a workgroup), token counts below,
# at and past the 16-wave shares, ragged channel counts, row strides past d
@pytest.mark.parametrize("cross", [False, True])
@pytest.mark.parametrize("n,d", [(1, 1), (3, 17), (130, 256), (2049, 257), (515, 530), (77, 1030),
                                 (1000, 1100), (129, 1601)])
def test_cov_fp32_tiles(n, d, cross):
    rng = np.random.default_rng(n * 7 + d)
    a = rng.standard_normal((n, d + 3)).astype(np.float32)
    b = rng.standard_normal((n, d + 3)).astype(np.float32) if cross else a
    h0 = rng.standard_normal((d, d)).astype(np.float32)
    A, B = torch.from_numpy(a).to(DEV)[:, :d], torch.from_numpy(b).to(DEV)[:, :d]
    note(f"cov fp32 n={n} d={d} cross={cross}")
    for beta in (0.0, 0.5):
        H = torch.from_numpy(h0).to(DEV) if beta else torch.full((d, d), float("nan"), device=DEV)
        ws = torch.empty(256, dtype=torch.uint8, device=DEV)
        if cross:
            K.kronq_accumulate_cross(A, B, H, 2.0, beta, ws)
        else:
            K.kronq_accumulate_cov(A, H, 2.0, beta, ws)
        torch.cuda.synchronize()
        ref = 2.0 * (a[:, :d].astype(np.float64).T @ b[:, :d].astype(np.float64)) + beta * h0
        # n-term fp32 sums of the products: n 2^-24 of the sum of the terms' sizes at most
        size = 2.0 * (np.abs(a[:, :d]).astype(np.float64).T @ np.abs(b[:, :d])) + np.abs(beta * h0)
        assert np.all(np.abs(to_np(H) - ref) <= (n + 4) * 2.0 ** -24 * size)
        if not cross and beta == 0.0:
            assert np.array_equal(to_np(H), to_np(H).T)
