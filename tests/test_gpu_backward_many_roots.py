"""2-hop backward calls of so many roots that a workgroup of 512 threads for each would be 2^32 threads, which a
launch cuts off without an error.  One leaf per slot, eight slots per root, so grad_x is a histogram of the leaves
weighted by grad_out (about 670 additions into an element, 1e-5 of their magnitudes)."""
import numpy as np
import pytest
import torch

from parity_util import assert_close, to_f64

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
B, K1, N = (1 << 23) + 1, 8, 100_000


@pytest.mark.parametrize("weighted", [False, True])
def test_more_roots_than_one_launch_takes(weighted):
    from paper_2511_13645_amd import binding as fsa
    gen = torch.Generator(device=DEV).manual_seed(1)
    ids1 = torch.zeros((B, K1), dtype=torch.int32, device=DEV)
    ids2 = torch.randint(0, N, (B, K1, 1), generator=gen, device=DEV, dtype=torch.int32)
    g = torch.randn((B, 1), generator=gen, device=DEV)
    gx = torch.zeros((N, 1), device=DEV)
    if weighted:                                                    # equal weights: the plain mean
        w = torch.full((B, K1), 0.5, device=DEV)
        fsa.fsa_wmean_bwd(g, ids1, w, ids2, w.view(B, K1, 1), grad_x=gx)
    else:
        fsa.fsa_mean_bwd(g, ids1, ids2, grad_x=gx)
    torch.cuda.synchronize()
    leaf = ids2.view(-1).cpu().numpy()
    w = np.repeat(to_f64(g)[:, 0] / K1, K1)
    want = np.bincount(leaf, weights=w, minlength=N)[:, None]
    mag = np.bincount(leaf, weights=np.abs(w), minlength=N)[:, None]
    assert_close(to_f64(gx), want, mag, 1e-5, "grad_x")
