"""1-hop backward with rows that the seeds of a workgroup share: more such rows than fit in LDS, rows of every
kind of remainder, and batches on both sides of the lines at which waves per workgroup and seeds per wave grow."""
import numpy as np
import pytest
import torch

from parity_util import assert_close, to_f64

pytestmark = pytest.mark.gpu

N = 4000


@pytest.fixture(scope="module")
def fsa():
    from paper_2511_13645_amd import binding
    binding.lib()
    return binding


def _ids(rng, B, k, shared):
    """Half of the IDs from `shared` rows, the others from anywhere; holes, parallel edges, a seed with nothing."""
    ids = np.where(rng.random((B, k)) < 0.5, rng.integers(0, shared, (B, k)) * (N // shared), rng.integers(0, N, (B, k)))
    ids = ids.astype(np.int32)
    ids[rng.random((B, k)) < 0.15] = -1
    if k > 1:
        ids[:, 1] = ids[:, 0]
    ids[B // 2] = -1
    return ids


@pytest.mark.parametrize("D", [3, 20, 64, 100, 128, 257, 602])
@pytest.mark.parametrize("B, k, shared", [(1, 5, 2), (5, 64, 40), (1025, 7, 300), (2049, 15, 3), (4097, 10, 60), (9001, 4, 500)])
def test_shared_rows(fsa, orc, B, k, shared, D):
    rng = np.random.default_rng(B + D)
    ids = _ids(rng, B, k, shared)
    w = rng.random((B, k)).astype(np.float32)
    w[0] = 0.0
    g = rng.standard_normal((B, D)).astype(np.float32)
    up = lambda a: torch.from_numpy(a).to("cuda:0")
    gx, wgx = torch.zeros((2, N, D), device="cuda:0")
    fsa.fsa_mean_bwd(up(g), up(ids), grad_x=gx)
    fsa.fsa_wmean_bwd(up(g), up(ids), up(w), grad_x=wgx)
    torch.cuda.synchronize()
    f64 = lambda a: a.astype(np.float64)
    # a row's sum of n additions in fp32, in any order, is within n * 2^-24 of sum |contribution|; 1e-5 covers n = 160
    adds = np.bincount(ids[ids >= 0], minlength=N).max()
    tol = max(1e-5, float(adds) * 2.0 ** -24)
    assert_close(to_f64(gx), orc.mean_bwd(f64(g), ids, num_nodes=N), orc.mean_bwd(f64(np.abs(g)), ids, num_nodes=N), tol, "grad_x")
    assert_close(to_f64(wgx), orc.wmean_bwd(f64(g), ids, w, num_nodes=N), orc.wmean_bwd(f64(np.abs(g)), ids, w, num_nodes=N), tol,
                 "weighted grad_x")


@pytest.mark.parametrize("dtype, step", [(torch.bfloat16, 2.0 ** -8), (torch.float16, 2.0 ** -10)])
@pytest.mark.parametrize("B, k, D", [(300, 6, 20), (2500, 5, 130), (9001, 3, 200)])
def test_shared_rows_16_bit(fsa, orc, dtype, step, B, k, D):
    rng = np.random.default_rng(B)
    ids = _ids(rng, B, k, 200)
    g = rng.standard_normal((B, D)).astype(np.float32)
    up = lambda a: torch.from_numpy(a).to("cuda:0")
    gx = torch.zeros((N, D), dtype=dtype, device="cuda:0")
    fsa.fsa_mean_bwd_lp(up(g), up(ids), grad_x=gx)
    torch.cuda.synchronize()
    ref = orc.mean_bwd(g.astype(np.float64), ids, num_nodes=N)
    mag = orc.mean_bwd(np.abs(g).astype(np.float64), ids, num_nodes=N)
    # every contribution is rounded once and each of the n additions rounds the running sum: n + 1 ulps
    adds = np.bincount(ids[ids >= 0], minlength=N)[:, None]
    bound = (adds + 1) * (step * mag + (2.0 ** -24 if dtype == torch.float16 else 2.0 ** -133))
    assert bool((np.abs(to_f64(gx) - ref) <= bound).all())


def _exact_ids(rng, B, k, width):
    """1, 2 or 4 live IDs per seed (or none), among holes, nearly all from the `width` rows that 32 seeds in a row share,
    some twice."""
    block = np.arange(B)[:, None] // 32
    ids = np.where(rng.random((B, k)) < 0.95, (block * 37 + rng.integers(0, width, (B, k)) * 5) % N, rng.integers(0, N, (B, k)))
    live = rng.choice([0, 1, 2, 4], B, p=[0.02, 0.04, 0.04, 0.9])
    twice = (live > 1) & (rng.random(B) < 0.3)
    ids[twice, 1] = ids[twice, 0]
    ids[np.arange(k) >= live[:, None]] = -1
    return rng.permuted(ids, axis=1).astype(np.int32)


# Gradients of 0 and +-4, and divisors of 1, 2 and 4: every contribution and every partial sum, in whatever order, is
# a whole number, and exact while it has no more bits than the type, which the test looks at.
@pytest.mark.parametrize("dtype, exact", [(torch.float32, 2.0 ** 24), (torch.bfloat16, 2.0 ** 8), (torch.float16, 2.0 ** 11)])
@pytest.mark.parametrize("units", [0, 1, 15])             # of 4 bytes: where grad_x starts in its 64-byte segment
@pytest.mark.parametrize("B, k, width, D", [(300, 6, 3, 20), (2500, 5, 12, 130), (4000, 7, 5, 200), (9001, 4, 28, 602)])
def test_shared_rows_to_the_last_bit(fsa, orc, B, k, width, D, units, dtype, exact):
    rng = np.random.default_rng(B + units)
    ids = _exact_ids(rng, B, k, width)
    g = rng.choice([-4.0, 0.0, 4.0], (B, D), p=[0.2, 0.6, 0.2])
    assert orc.mean_bwd(np.abs(g), ids, num_nodes=N).max() <= exact
    up = lambda a: torch.from_numpy(a).to("cuda:0")
    start = 64 + units * (1 if dtype == torch.float32 else 2)
    buf = torch.ones(start + N * D + 64, dtype=dtype, device="cuda:0")
    assert buf.data_ptr() % 64 == 0
    gx = buf[start:start + N * D].view(N, D)
    gx.zero_()
    fsa.fsa_mean_bwd_lp(up(g.astype(np.float32)), up(ids), grad_x=gx)
    torch.cuda.synchronize()
    assert np.array_equal(to_f64(gx), orc.mean_bwd(g, ids, num_nodes=N))
    assert bool((buf[:start] == 1).all()) and bool((buf[start + N * D:] == 1).all())
