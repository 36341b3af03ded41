"""The backward into a gradient of its own (fsa_mean_bwd_dense) against the oracle: rows that nothing names, bins and
rows that end anywhere, hub rows beyond a bin's room, holes, and nothing written outside the table."""
import numpy as np
import pytest
import torch

from parity_util import assert_close, to_f64

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
# fp32: sums of fp32 terms (the other backwards' bound); 16 bits: the same sum rounded, by 2^-8 or 2^-11 at most, once per
# 256 leaves of the row's bin (the hub's row is the only one here whose bin has more than 256)
TOL = {torch.float32: 1e-5, torch.bfloat16: 2.0 ** -8 + 1e-5, torch.float16: 2.0 ** -11 + 1e-5}


def _ids(rng, n, B, k1, k2, hub):
    ids1 = rng.integers(0, n, (B, k1)).astype(np.int32)
    ids1[rng.random((B, k1)) < 0.2] = -1
    ids2 = None
    if k2:
        ids2 = rng.integers(0, n, (B, k1, k2)).astype(np.int32)
        ids2[rng.random((B, k1, k2)) < 0.2] = -1
    leaf = ids1 if ids2 is None else ids2
    leaf[(rng.random(leaf.shape) < hub) & (leaf >= 0)] = n // 3         # one row named most often
    return ids1, ids2


@pytest.mark.parametrize("n,D,B,k1,k2,dtype,slot_grads,hub", [
    (1, 1, 1, 1, 0, torch.float32, False, 0.0),
    (2000, 128, 300, 15, 10, torch.float32, False, 0.05),
    (2000, 128, 300, 15, 10, torch.float32, True, 0.05),
    (5001, 37, 257, 7, 3, torch.float32, True, 0.3),                   # odd rows, a last bin that is not full
    (5001, 300, 64, 64, 5, torch.float32, False, 0.9),                 # a bin far beyond its room
    (70001, 17, 9, 3, 2, torch.float32, True, 0.0),                    # nearly every bin empty, many counters
    (999, 1024, 40, 5, 4, torch.float32, True, 0.1),                   # the widest row, eight to a bin
    (1000, 64, 1024, 10, 0, torch.float32, False, 0.1),
    (777, 5, 1001, 64, 0, torch.float32, False, 0.5),
    (2000, 128, 300, 15, 10, torch.bfloat16, True, 0.05),
    (3003, 33, 130, 6, 64, torch.float16, True, 0.1),
    (3003, 601, 130, 25, 0, torch.bfloat16, False, 0.1),
])
def test_dense_backward_matches_the_oracle(orc, n, D, B, k1, k2, dtype, slot_grads, hub):
    from paper_2511_13645_amd import binding
    rng = np.random.default_rng(n + D)
    ids1, ids2 = _ids(rng, n, B, k1, k2, hub)
    d = lambda a: None if a is None else torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    g = d(rng.standard_normal((B, D)).astype(np.float32)).to(dtype)
    gh = d(rng.standard_normal((B, k1, D)).astype(np.float32)).to(dtype) if slot_grads else None
    need = binding.fsa_mean_bwd_dense_workspace_bytes(B, k1, k2, D, n)
    assert need > 0
    ws = torch.full((need,), 0xA5, dtype=torch.uint8, device=DEV)
    whole = torch.full((n * D + 4096,), float("nan"), dtype=dtype, device=DEV)
    for _ in range(2):                                                  # the second call finds the first one's workspace
        binding.fsa_mean_bwd_dense(g, d(ids1), d(ids2), gh, grad_x=whole[:n * D].view(n, D), workspace=ws)
    torch.cuda.synchronize()
    assert torch.isnan(whole[n * D:]).all()
    ref = orc.mean_bwd(to_f64(g), ids1, ids2, None if gh is None else to_f64(gh), num_nodes=n)
    scale = orc.mean_bwd(np.abs(to_f64(g)), ids1, ids2, None if gh is None else np.abs(to_f64(gh)), num_nodes=n)
    if dtype != torch.float32:
        leaf = ids1 if ids2 is None else np.where(ids1[..., None] >= 0, ids2, -1)
        per_row = np.bincount(leaf[leaf >= 0].ravel(), minlength=n)
        near = max(32, min(256, 8192 // D))                              # rows that can share a bin with it
        in_bin = np.convolve(per_row, np.ones(2 * near + 1, dtype=np.int64), "same")
        scale = scale * (1 + in_bin // 256 + (in_bin > 256))[:, None]
    # fp16: results below the smallest normal number are spaced 2^-24
    assert_close(to_f64(whole[:n * D].view(n, D)), ref, scale + (2.0 ** -12 if dtype == torch.float16 else 0.0), TOL[dtype],
                 "dense backward n=%d D=%d" % (n, D))


def test_dense_backward_refuses_what_it_cannot_take():
    from paper_2511_13645_amd import binding
    n, D, B, k1 = 100, 8, 4, 3
    g = torch.zeros((B, D), device=DEV)
    ids1 = torch.zeros((B, k1), dtype=torch.int32, device=DEV)
    need = binding.fsa_mean_bwd_dense_workspace_bytes(B, k1, 0, D, n)
    ws = torch.empty(need + 256, dtype=torch.uint8, device=DEV)
    x = torch.empty(n * D + 4, device=DEV)
    for bad in (dict(workspace=ws[:need - 1]), dict(workspace=ws[16:16 + need]), dict(grad_x=x[1:1 + n * D].view(n, D))):
        with pytest.raises(binding.FsaError):
            binding.fsa_mean_bwd_dense(g, ids1, **{**dict(grad_x=x[:n * D].view(n, D), workspace=ws[:need]), **bad})
    with pytest.raises((TypeError, ValueError)):
        binding.fsa_mean_bwd_dense(g, ids1, grad_x=x[:n * D].view(n, D).half(), workspace=ws)
    assert binding.fsa_mean_bwd_dense_workspace_bytes(B, k1, 0, 1025, n) == 0
    assert binding.fsa_mean_bwd_dense_workspace_bytes(0, k1, 0, D, n) == 0


def test_autograd_takes_the_dense_route_and_replays_in_a_graph(orc):
    from paper_2511_13645_amd import binding
    from paper_2511_13645_amd.autograd import fused_sample_mean
    n, D, B, fan = 20000, 64, 1024, [25, 10]
    rng = np.random.default_rng(5)
    deg = rng.integers(0, 30, size=n)
    indptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    indices = (n * rng.random(int(indptr[-1])) ** 3).astype(np.int32)      # some rows named often
    assert binding.fsa_mean_bwd_dense_pays(B, fan[0], fan[1], D, torch.float32, n)
    d = lambda a: torch.from_numpy(a).to(DEV)
    x = torch.nn.Parameter(torch.randn((n, D), device=DEV))
    g = torch.randn((B, D), device=DEV)
    args = d(indptr), d(indices), d(rng.integers(0, n, B).astype(np.int32)), fan, 7

    def step():
        x.grad = None
        out, _, ids1, ids2 = fused_sample_mean(x, *args)
        out.backward(g)
        return ids1, ids2
    ids1, ids2 = step()
    a1, a2 = ids1.cpu().numpy(), ids2.cpu().numpy()
    ref = orc.mean_bwd(to_f64(g), a1, a2, None, num_nodes=n)
    scale = orc.mean_bwd(np.abs(to_f64(g)), a1, a2, None, num_nodes=n)
    assert_close(to_f64(x.grad), ref, scale, 1e-5, "autograd, dense route")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step()
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    x.grad = None
    with torch.cuda.graph(graph):
        step()
    captured = x.grad
    for _ in range(3):
        captured.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert_close(to_f64(captured), ref, scale, 1e-5, "autograd, dense route, replayed")


@pytest.mark.parametrize("short_of_memory", [False, True])
def test_dense_gradient_through_python_and_without_room_for_its_workspace(monkeypatch, short_of_memory):
    from paper_2511_13645_amd import binding
    n, D, B, k1, k2 = 20000, 64, 1024, 25, 10
    gen = torch.Generator(device=DEV).manual_seed(3)
    ids1 = torch.randint(0, n, (B, k1), generator=gen, device=DEV, dtype=torch.int32)
    ids2 = torch.randint(0, n, (B, k1, k2), generator=gen, device=DEV, dtype=torch.int32)
    g = torch.randn((B, D), generator=gen, device=DEV)
    native = binding.grad_dense(g, ids1, ids2, None, n)
    monkeypatch.setattr(binding, "_host", None)
    if short_of_memory:
        def none_left(*a, **kw):
            raise torch.cuda.OutOfMemoryError("no memory")
        monkeypatch.setattr(binding, "fsa_mean_bwd_dense_workspace_bytes", none_left)
        assert binding.grad_dense(g, ids1, ids2, None, n) is None
    else:
        # two orders of up to a few dozen fp32 additions a row
        assert torch.allclose(binding.grad_dense(g, ids1, ids2, None, n), native, rtol=1e-5, atol=1e-6)
    assert binding.grad_dense(g[:1], ids1[:1], ids2[:1], None, n) is None      # too small to pay
