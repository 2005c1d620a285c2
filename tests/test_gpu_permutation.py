"""Permutations on both sides of the sizes where the buckets change, bit for bit against the oracle."""
import numpy as np
import pytest
import torch

from gpu_util import host
from oracle import rng as orng

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [7, 8, 15, 16, 17, 262143, 262144, 524289, 33554431, 33554432])
def test_permutation_bucket_edges(B):
    import paper_2509_10771_amd as rx
    rx.rslx_device_check()
    out = torch.full((B,), -1, dtype=torch.int32, device="cuda")
    rx.rslx_permutation(5, 2, 1, B, out, rx.workspace(rx.rslx_permutation_workspace_bytes(B)))
    torch.cuda.synchronize()
    assert np.array_equal(host(out), orng.permutation(5, 2, 1, B))
