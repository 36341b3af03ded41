"""Atomic 2-hop backwards on rows that start anywhere in a 64-byte segment, rows narrow enough to share an
instruction, and roots whose leaves several workgroups share out: against the oracle, with the bytes around
grad_x untouched."""
import numpy as np
import pytest
import torch

from parity_util import assert_close, to_f64

pytestmark = pytest.mark.gpu

N, K1, K2 = 700, 5, 9
GUARD = 64                                     # elements before and after grad_x


@pytest.fixture(scope="module")
def fsa():
    from paper_2511_13645_amd import binding
    binding.lib()
    return binding


def _ids(rng, B, distinct=False):
    if distinct:                               # every row at most once in the call
        flat = np.full(B * K1 * K2, -1, np.int32)
        at = rng.permutation(flat.size)[:min(N, flat.size)]
        flat[at] = rng.permutation(N)[:at.size]
        ids2 = flat.reshape(B, K1, K2)
    else:
        ids2 = rng.integers(0, N, (B, K1, K2)).astype(np.int32)
        ids2[rng.random(ids2.shape) < 0.2] = -1
        ids2[:, :, 1] = ids2[:, :, 0]          # parallel edges
    ids1 = rng.integers(0, N, (B, K1)).astype(np.int32)
    ids1[rng.random(ids1.shape) < 0.1] = -1
    ids2[ids1 < 0] = -1
    return ids1, ids2


def _grad_x(D, dtype, offset):
    """grad_x [N,D] of zeros inside a buffer of ones, `offset` elements past a 64-byte boundary."""
    buf = torch.ones(2 * GUARD + offset + N * D, dtype=dtype, device="cuda:0")
    assert buf.data_ptr() % 64 == 0
    gx = buf[GUARD + offset:GUARD + offset + N * D].view(N, D)
    gx.zero_()
    return buf, gx


def _guards_intact(buf, D, offset):
    return bool((buf[:GUARD + offset] == 1).all()) and bool((buf[GUARD + offset + N * D:] == 1).all())


# rows of one segment, two, one instruction, and of several with every kind of remainder; B: leaves shared out
# by several workgroups, or one workgroup a root
@pytest.mark.parametrize("B", [1, 70, 300])
@pytest.mark.parametrize("offset", [0, 1, 15])
@pytest.mark.parametrize("D", [1, 15, 16, 17, 32, 33, 49, 64, 65, 79, 80, 100, 113, 128, 129, 602])
def test_fp32_rows(fsa, orc, D, offset, B):
    rng = np.random.default_rng(D * 131 + offset * 7 + B)
    ids1, ids2 = _ids(rng, B)
    w1 = rng.random((B, K1)).astype(np.float32)
    w2 = rng.random((B, K1, K2)).astype(np.float32)
    g = rng.standard_normal((B, D)).astype(np.float32)
    gh = rng.standard_normal((B, K1, D)).astype(np.float32)
    up = lambda a: torch.from_numpy(a).to("cuda:0")
    buf, gx = _grad_x(D, torch.float32, offset)
    fsa.fsa_mean_bwd(up(g), up(ids1), up(ids2), up(gh), grad_x=gx)
    wbuf, wgx = _grad_x(D, torch.float32, offset)
    fsa.fsa_wmean_bwd(up(g), up(ids1), up(w1), up(ids2), up(w2), up(gh), grad_x=wgx)
    torch.cuda.synchronize()
    f64 = lambda a: a.astype(np.float64)
    ref = orc.mean_bwd(f64(g), ids1, ids2, f64(gh), num_nodes=N)
    mag = orc.mean_bwd(f64(np.abs(g)), ids1, ids2, f64(np.abs(gh)), num_nodes=N)
    assert_close(to_f64(gx), ref, mag, 1e-5, "grad_x")
    ref = orc.wmean_bwd(f64(g), ids1, w1, ids2, w2, f64(gh), num_nodes=N)
    mag = orc.wmean_bwd(f64(np.abs(g)), ids1, w1, ids2, w2, f64(np.abs(gh)), num_nodes=N)
    assert_close(to_f64(wgx), ref, mag, 1e-5, "weighted grad_x")
    assert _guards_intact(buf, D, offset) and _guards_intact(wbuf, D, offset)


# 16-bit rows: every row receives one contribution, so the result is the fp32 call's, rounded once
@pytest.mark.parametrize("B", [2, 300])
@pytest.mark.parametrize("offset", [0, 2, 30])
@pytest.mark.parametrize("D", [2, 32, 34, 64, 66, 128, 130, 200, 330])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
def test_16_bit_rows(fsa, dtype, D, offset, B):
    rng = np.random.default_rng(D * 17 + offset + B)
    ids1, ids2 = _ids(rng, B, distinct=True)
    up = lambda a: torch.from_numpy(a).to("cuda:0")
    g = up(rng.standard_normal((B, D)).astype(np.float32))
    want = torch.zeros((N, D), device="cuda:0")
    fsa.fsa_mean_bwd(g, up(ids1), up(ids2), grad_x=want)
    buf, gx = _grad_x(D, dtype, offset)
    fsa.fsa_mean_bwd_lp(g, up(ids1), up(ids2), grad_x=gx)
    torch.cuda.synchronize()
    normal = want.abs() >= torch.finfo(dtype).tiny     # an atomic may flush a 16-bit subnormal
    assert torch.equal(gx[normal], want.to(dtype)[normal])
    assert bool((gx[~normal].float().abs() <= torch.finfo(dtype).tiny).all())
    assert _guards_intact(buf, D, offset)
