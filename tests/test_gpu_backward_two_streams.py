"""Backward calls without a workspace add atomically, so calls on two streams may fill one gradient table
at the same time.  Sizes at which a workspace would switch to plain loads and stores, few rows, so that
the streams meet on them; the sum must be that of both calls (1e-5 of the contributions' magnitudes)."""
import numpy as np
import pytest
import torch

from parity_util import assert_close, marked_workspace, to_f64, workspace_route
from test_gpu_backward_workspace import _ids

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
B, K1, K2, K3, D, N = 1400, 10, 10, 3, 128, 1500


@pytest.fixture(scope="module")
def fsa():
    from paper_2511_13645_amd import binding
    binding.lib()
    return binding


def _inputs(seed):
    rng = np.random.default_rng(seed)
    ids1, ids2 = _ids(rng, B, K1, K2, N)
    ids3 = rng.integers(-1, N, (B, K1, K2, K3)).astype(np.int32)
    f = lambda *s: torch.from_numpy(rng.random(s, dtype=np.float32)).to(DEV)
    return {"g": f(B, D) - 0.5, "gh": f(B, K1, D) - 0.5, "w1": f(B, K1), "w2": f(B, K1, K2),
            **{k: torch.from_numpy(v).to(DEV) for k, v in (("i1", ids1), ("i2", ids2), ("i3", ids3))}}


CALLS = {
    "fsa_mean_bwd": lambda fsa, c, gx: fsa.fsa_mean_bwd(c["g"], c["i1"], c["i2"], c["gh"], grad_x=gx),
    "fsa_mean_bwd_ws without a workspace": lambda fsa, c, gx: fsa.fsa_mean_bwd_ws(c["g"], c["i1"], c["i2"], c["gh"], grad_x=gx),
    "fsa_mean_bwd_lp": lambda fsa, c, gx: fsa.fsa_mean_bwd_lp(c["g"], c["i1"], c["i2"], c["gh"], grad_x=gx),
    "fsa_wmean_bwd": lambda fsa, c, gx: fsa.fsa_wmean_bwd(c["g"], c["i1"], c["w1"], c["i2"], c["w2"], c["gh"], grad_x=gx),
    "fsa_mean3_bwd": lambda fsa, c, gx: fsa.fsa_mean3_bwd(c["g"], c["i1"], c["i2"], c["i3"], grad_h1=c["gh"], grad_x=gx),
}


@pytest.mark.parametrize("name", CALLS)
def test_two_streams_fill_one_table(fsa, name):
    call = CALLS[name]
    assert fsa.fsa_bwd_workspace_bytes(B, K1, K2, D) > 0
    pair = [_inputs(1), _inputs(2)]
    want, mag = np.zeros((N, D)), np.zeros((N, D))
    for c in pair:                                         # one after the other, into tables of their own
        want += to_f64(call(fsa, c, torch.zeros((N, D), device=DEV)))
        mag += to_f64(call(fsa, {**c, "g": c["g"].abs(), "gh": c["gh"].abs()}, torch.zeros((N, D), device=DEV)))
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for _ in range(3):
        gx = torch.zeros((N, D), device=DEV)
        torch.cuda.synchronize()
        for s, c in zip(streams, pair):
            with torch.cuda.stream(s):
                call(fsa, c, gx)
        torch.cuda.synchronize()
        assert_close(to_f64(gx), want, mag, 1e-5, name)


def test_two_forwards_on_two_streams_share_a_master_gradient(fsa):
    from paper_2511_13645_amd.autograd import fused_sample_mean
    rng = np.random.default_rng(3)
    n = N
    deg = rng.integers(20, 60, n)
    indptr = torch.from_numpy(np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)).to(DEV)
    indices = torch.from_numpy(rng.integers(0, n, int(deg.sum())).astype(np.int32)).to(DEV)
    x = torch.randn((n, D), device=DEV).to(torch.bfloat16).requires_grad_(True)
    seeds = [torch.from_numpy(rng.integers(0, n, B).astype(np.int32)).to(DEV) for _ in range(2)]
    grads = [torch.randn((B, D), device=DEV).to(torch.bfloat16) for _ in range(2)]
    torch.cuda.synchronize()

    def fill(streams, sign):
        master = torch.zeros((n, D), device=DEV)
        torch.cuda.synchronize()
        outs = []
        for s, st in zip(seeds, streams):
            with torch.cuda.stream(st):
                outs.append(fused_sample_mean(x, indptr, indices, s, [K1, K2], 5, master_grad=master)[0])
        torch.autograd.backward(outs, [g.abs() if sign else g for g in grads])
        torch.cuda.synchronize()
        return to_f64(master)

    one = torch.cuda.current_stream()
    assert_close(fill([torch.cuda.Stream(), torch.cuda.Stream()], False), fill([one, one], False), fill([one, one], True), 1e-5, "master_grad")


def test_a_kept_workspace_leaves_calls_outside_the_sorted_route_to_atomics(fsa):
    """fsa_mean_bwd_ws takes its one route for the shapes that fsa_mean_bwd_workspace_bytes names, whatever the workspace."""
    assert fsa.fsa_mean_bwd_workspace_bytes(B, K1, K2, D) == 0
    ws = marked_workspace(64 << 20)
    c = _inputs(4)
    gx = torch.zeros((N, D), device=DEV)
    fsa.fsa_mean_bwd_ws(c["g"], c["i1"], c["i2"], grad_x=gx, workspace=ws)
    torch.cuda.synchronize()
    assert workspace_route(ws) == "atomic"
