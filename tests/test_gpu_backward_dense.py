"""The backward into a gradient of its own (fsa_mean_bwd_dense) against the oracle: rows that nothing names, bins and
rows that end anywhere, hub rows beyond a bin's room, holes, and nothing written outside the table."""
import numpy as np
import pytest
import torch

from parity_util import assert_close, marked_workspace, to_f64, workspace_route

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
# fp32: sums of fp32 terms (the other backwards' bound); 16 bits: the same sum rounded, by 2^-8 or 2^-11 at most, once per
# 256 leaves of the row's bin (_roundings)
TOL = {torch.float32: 1e-5, torch.bfloat16: 2.0 ** -8 + 1e-5, torch.float16: 2.0 ** -11 + 1e-5}


def _roundings(ids1, ids2, n, D):
    """How often a 16-bit row is rounded at most, [n,1]: a bin is a run of rows that starts at a multiple of its length, this
    one or a half, a quarter ... of it."""
    rows = 256
    while rows > 32 and rows * D > 8192:
        rows //= 2
    leaf = ids1 if ids2 is None else np.where(ids1[..., None] >= 0, ids2, -1)
    in_bin = np.bincount(leaf[leaf >= 0].ravel() // rows, minlength=-(-n // rows))
    return np.maximum(1, -(-in_bin // 256)).repeat(rows)[:n, None]


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


@pytest.mark.parametrize("n,D,B,k1,k2,dtype,slot_grads,hub,single_rounding", [
    (1, 1, 1, 1, 0, torch.float32, False, 0.0, None),
    (2000, 128, 300, 15, 10, torch.float32, False, 0.05, None),
    (2000, 128, 300, 15, 10, torch.float32, True, 0.05, None),
    (5001, 37, 257, 7, 3, torch.float32, True, 0.3, None),             # odd rows, a last bin that is not full
    (5001, 300, 64, 64, 5, torch.float32, False, 0.9, None),           # a bin far beyond its room
    (70001, 17, 9, 3, 2, torch.float32, True, 0.0, None),              # nearly every bin empty, many counters
    (999, 1024, 40, 5, 4, torch.float32, True, 0.1, None),             # the widest row, 32 to a bin
    (1000, 64, 1024, 10, 0, torch.float32, False, 0.1, None),
    (777, 5, 1001, 64, 0, torch.float32, False, 0.5, None),            # every bin beyond its room
    (40000, 12, 2500, 3, 2, torch.float32, True, 0.02, None),          # workgroups of the binning that take many roots
    (150, 20, 40, 64, 64, torch.float32, True, 0.2, None),             # and of one root of 4096 leaf slots
    (301, 37, 3000, 16, 12, torch.float32, True, 0.3, None),           # lists of more entries than are shared out at once,
    (300, 12, 6000, 64, 0, torch.float32, False, 0.02, None),          # with a hub and without
    (20000, 128, 300, 15, 10, torch.bfloat16, True, 0.0, True),
    (20011, 33, 300, 6, 3, torch.float16, True, 0.0, True),
    (2000, 128, 300, 15, 10, torch.bfloat16, True, 0.05, False),
    (3003, 33, 130, 6, 64, torch.float16, True, 0.1, False),
    (3003, 601, 130, 25, 0, torch.bfloat16, False, 0.1, False),
    (777, 5, 1001, 64, 0, torch.bfloat16, False, 0.5, False),
])
def test_dense_backward_matches_the_oracle(orc, n, D, B, k1, k2, dtype, slot_grads, hub, single_rounding):
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
        roundings = _roundings(ids1, ids2, n, D)
        assert single_rounding is None or (roundings.max() == 1) == single_rounding
        scale = scale * roundings
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


def test_16bit_rows_of_full_bins_are_rounded_once_in_256_entries():
    """Every bin holds far more entries than it has room for.  A row of m equal terms, whose sum is exact in fp32, is off
    by half a unit in the last place of the running sum for each rounding, and there is one per 256 entries of its bin; a
    row rounded at every addition would stop growing at 256 terms."""
    from paper_2511_13645_amd import binding
    n, D, B, k1 = 2048, 256, 48000, 64                                  # 32 rows to a bin, about 48,000 entries in each
    rows_of_bin = 32
    gen = torch.Generator(device=DEV).manual_seed(11)
    ids1 = torch.randint(0, n, (B, k1), generator=gen, device=DEV, dtype=torch.int32)
    g = torch.ones((B, D), dtype=torch.bfloat16, device=DEV)
    ws = torch.empty(binding.fsa_mean_bwd_dense_workspace_bytes(B, k1, 0, D, n), dtype=torch.uint8, device=DEV)
    grad = binding.fsa_mean_bwd_dense(g, ids1, grad_x=torch.empty((n, D), dtype=torch.bfloat16, device=DEV), workspace=ws)
    terms = torch.bincount(ids1.flatten(), minlength=n).double().cpu().numpy()
    roundings = int(1.05 * B * k1 / (n // rows_of_bin) / 256)            # (bins differ by 0.5 %)
    # the i-th of r roundings meets a sum of about i/r of the whole: half a unit is 2^-8 of the power of two below it
    sums = (terms / k1)[:, None] * (np.arange(1, roundings + 1) / roundings)
    bound = (2.0 ** (np.floor(np.log2(sums)) - 8)).sum(1)
    err = np.abs(to_f64(grad) - (terms / k1)[:, None]).max(1)
    assert (err <= bound).all(), (err / bound).max()
    assert bound.max() < 0.5 * (terms / k1).max()                       # and the bound says something


def _skewed(name, n, shape):
    """Leaf IDs, none of them a hole: `hub` a tenth on one row, `star` all, `front` nine tenths on the first hundredth."""
    gen = torch.Generator(device=DEV).manual_seed(7)
    leaf = torch.randint(0, n, shape, generator=gen, device=DEV, dtype=torch.int32)
    if name == "front":
        leaf = torch.where(torch.rand(shape, generator=gen, device=DEV) < 0.9, leaf // 100, leaf)
    if name == "star":
        leaf.fill_(n // 2)
    if name == "hub":
        leaf[torch.rand(shape, generator=gen, device=DEV) < 0.1] = n // 2
    return leaf


def _least_us(call, turns=7):
    """Least time of a call on the GPU, the queue being full."""
    call()
    best = float("inf")
    for _ in range(turns):
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda._sleep(1_000_000)                                    # the host is ahead when the timed part starts
        start.record()
        call()
        end.record()
        end.synchronize()
        best = min(best, start.elapsed_time(end) * 1e3)
    return best


# Batches that once took 2 to 100 times as long on this route as clearing and adding with atomics, the last one half as long
# again, and now take less time or, the last one, the same: a bound half-way between, far from what runs of either differ by.
@pytest.mark.parametrize("skew,n,D,B,k1,k2", [
    ("hub", 50000, 1000, 1024, 15, 10),
    ("star", 100000, 128, 1024, 15, 10),
    ("hub", 200000, 20, 4096, 15, 10),
    ("even", 20000, 64, 5000, 25, 10),
    ("even", 10000, 64, 8192, 15, 10),
    ("front", 20000, 128, 2048, 25, 10),
    ("front", 100000, 128, 1024, 15, 10),
])
def test_skewed_batches_are_not_slower_than_clearing_and_adding(skew, n, D, B, k1, k2):
    from paper_2511_13645_amd import binding
    ids2 = _skewed(skew, n, (B, k1, k2))
    ids1 = torch.zeros((B, k1), dtype=torch.int32, device=DEV)
    g = torch.randn((B, D), generator=torch.Generator(device=DEV).manual_seed(8), device=DEV)
    grad = torch.empty((n, D), device=DEV)
    ws = torch.empty(binding.fsa_mean_bwd_dense_workspace_bytes(B, k1, k2, D, n), dtype=torch.uint8, device=DEV)
    dense = _least_us(lambda: binding.fsa_mean_bwd_dense(g, ids1, ids2, grad_x=grad, workspace=ws))
    added = _least_us(lambda: binding.fsa_mean_bwd(g, ids1, ids2, grad_x=grad.zero_()))
    assert dense <= 1.3 * added, "%.0f us against %.0f" % (dense, added)


@pytest.mark.parametrize("workspace", [lambda: torch.empty(1 << 20, dtype=torch.uint8),
                                       lambda: torch.empty((1 << 10, 1 << 10), dtype=torch.uint8, device=DEV).t()])
def test_autograd_refuses_what_is_no_workspace_on_every_route(workspace):
    """A host tensor and one that is not contiguous, with a call for the dense route and one for the atomics."""
    from paper_2511_13645_amd import binding
    from paper_2511_13645_amd.autograd import fused_sample_mean
    n, D, fan = 20000, 64, [25, 10]
    assert binding.fsa_mean_bwd_workspace_bytes(1024, *fan, D) == 0    # else the sorted route takes the call
    indptr = torch.arange(0, 5 * n + 1, 5, dtype=torch.int32, device=DEV)
    indices = torch.randint(0, n, (5 * n,), dtype=torch.int32, device=DEV)
    for B in (1024, 8):
        assert binding.fsa_mean_bwd_dense_pays(B, *fan, D, torch.float32, n) == (B > 8)
        x = torch.nn.Parameter(torch.randn((n, D), device=DEV))
        seeds = torch.arange(B, dtype=torch.int32, device=DEV)
        out, _, _, _ = fused_sample_mean(x, indptr, indices, seeds, fan, 1, workspace=workspace())
        with pytest.raises(ValueError):
            out.sum().backward()
        assert x.grad is None


def test_gradients_off_a_quads_alignment_give_the_same(orc):
    """Rows of whole quads at an odd address: one element a lane instead of four."""
    from paper_2511_13645_amd import binding
    n, D, B, k1, k2 = 3000, 64, 200, 6, 5
    rng = np.random.default_rng(4)
    ids1, ids2 = _ids(rng, n, B, k1, k2, 0.2)
    off = lambda *shape: torch.randn(int(np.prod(shape)) + 1, device=DEV)[1:].view(shape)
    g, gh = off(B, D), off(B, k1, D)
    assert g.data_ptr() % 16 == 4 and gh.data_ptr() % 16 == 4
    ws = torch.empty(binding.fsa_mean_bwd_dense_workspace_bytes(B, k1, k2, D, n), dtype=torch.uint8, device=DEV)
    d = lambda a: torch.from_numpy(a).to(DEV)
    got = binding.fsa_mean_bwd_dense(g, d(ids1), d(ids2), gh, grad_x=torch.empty((n, D), device=DEV), workspace=ws)
    ref = orc.mean_bwd(to_f64(g), ids1, ids2, to_f64(gh), num_nodes=n)
    scale = orc.mean_bwd(np.abs(to_f64(g)), ids1, ids2, np.abs(to_f64(gh)), num_nodes=n)
    assert_close(to_f64(got), ref, scale, 1e-5, "gradients off alignment")


def _table_case(n, D, B, dtype, seed, skew=3):
    """A graph, a table and seeds of two hops with fanouts 25 and 10; with a skew some rows are named often."""
    rng = np.random.default_rng(seed)
    deg = rng.integers(0, 30, size=n)
    indptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    indices = (n * rng.random(int(indptr[-1])) ** skew).astype(np.int32)
    d = lambda a: torch.from_numpy(a).to(DEV)
    x = torch.nn.Parameter(torch.randn((n, D), device=DEV).to(dtype))
    return x, (d(indptr), d(indices), d(rng.integers(0, n, B).astype(np.int32)), [25, 10], 7)


@pytest.mark.parametrize("native", [True, False])
@pytest.mark.parametrize("dtype,D", [(torch.float32, 64), (torch.bfloat16, 128), (torch.float16, 128)])
@pytest.mark.parametrize("outputs", ["out", "both", "h1"])
def test_autograd_on_the_dense_route_in_every_form(orc, monkeypatch, native, dtype, D, outputs):
    from paper_2511_13645_amd import binding
    from paper_2511_13645_amd.autograd import fused_sample_mean
    n, B = 20000, 1024
    x, args = _table_case(n, D, B, dtype, 6)
    assert binding.fsa_mean_bwd_dense_pays(B, 25, 10, D, dtype, n)
    if not native:
        monkeypatch.setattr(binding, "_host", None)

    def other(*a, **kw):
        raise AssertionError("the other route")
    monkeypatch.setattr(binding, "fsa_mean_bwd_ws", other)
    monkeypatch.setattr(binding, "fsa_mean_bwd_lp", other)
    out, h1, ids1, ids2 = fused_sample_mean(x, *args, want_h1=outputs != "out")
    g = torch.randn((B, D), device=DEV).to(dtype) if outputs != "h1" else torch.zeros((B, D), dtype=dtype, device=DEV)
    gh = torch.randn((B, 25, D), device=DEV).to(dtype) if outputs != "out" else None
    torch.autograd.backward([t for t, w in ((out, "h1"), (h1, "out")) if outputs != w], [t for t, w in ((g, "h1"), (gh, "out")) if outputs != w])
    a1, a2 = ids1.cpu().numpy(), ids2.cpu().numpy()
    ref = orc.mean_bwd(to_f64(g), a1, a2, None if gh is None else to_f64(gh), num_nodes=n)
    scale = orc.mean_bwd(np.abs(to_f64(g)), a1, a2, None if gh is None else np.abs(to_f64(gh)), num_nodes=n)
    if dtype != torch.float32:
        scale = scale * _roundings(a1, a2, n, D)
    assert x.grad.dtype == dtype
    assert_close(to_f64(x.grad), ref, scale + (2.0 ** -12 if dtype == torch.float16 else 0.0), TOL[dtype], "autograd, %s" % outputs)


@pytest.mark.parametrize("with_workspace", [True, False])
def test_a_workspace_of_the_sorted_route_keeps_autograd_on_it(orc, with_workspace):
    """Where fsa_mean_bwd_workspace_bytes asks for one: its sums have a fixed order, so two passes agree to the last bit."""
    from paper_2511_13645_amd import binding
    from paper_2511_13645_amd.autograd import fused_sample_mean
    n, D, B = 20000, 512, 1024
    x, args = _table_case(n, D, B, torch.float32, 9, skew=1)
    need = binding.fsa_mean_bwd_workspace_bytes(B, 25, 10, D)
    assert need > 0 and binding.fsa_mean_bwd_dense_pays(B, 25, 10, D, torch.float32, n)
    ws = marked_workspace(need)
    g = torch.randn((B, D), device=DEV)
    grads = []
    for _ in range(2):
        x.grad = None
        out, _, ids1, ids2 = fused_sample_mean(x, *args, workspace=ws if with_workspace else None)
        out.backward(g)
        grads.append(x.grad)
    assert workspace_route(ws) == ("sorted" if with_workspace else "atomic")    # "atomic": nobody wrote to it
    if with_workspace:
        assert torch.equal(*grads)
    a1, a2 = ids1.cpu().numpy(), ids2.cpu().numpy()
    ref = orc.mean_bwd(to_f64(g), a1, a2, None, num_nodes=n)
    scale = orc.mean_bwd(np.abs(to_f64(g)), a1, a2, None, num_nodes=n)
    assert_close(to_f64(grads[1]), ref, scale, 1e-5, "autograd with a workspace")


@pytest.mark.parametrize("native", [True, False])
def test_without_memory_for_the_workspace_the_gradient_is_cleared_and_added_to(monkeypatch, native):
    """The allocator's limit leaves room for the gradient and not for the workspace beside it."""
    from paper_2511_13645_amd import binding
    n, D, B, k1, k2 = 400000, 128, 2048, 25, 10
    gen = torch.Generator(device=DEV).manual_seed(3)
    ids1 = torch.randint(0, n, (B, k1), generator=gen, device=DEV, dtype=torch.int32)
    ids2 = torch.randint(0, n, (B, k1, k2), generator=gen, device=DEV, dtype=torch.int32)
    g = torch.randn((B, D), generator=gen, device=DEV)
    grad_bytes, need = n * D * 4, binding.fsa_mean_bwd_dense_workspace_bytes(B, k1, k2, D, n)
    assert binding.fsa_mean_bwd_dense_pays(B, k1, k2, D, torch.float32, n) and need > 48 << 20
    if not native:
        monkeypatch.setattr(binding, "_host", None)
    total = torch.cuda.get_device_properties(DEV).total_memory
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    held, limit = [], torch.cuda.memory_reserved()
    torch.cuda.set_per_process_memory_fraction(limit / total)
    try:
        with pytest.raises(torch.cuda.OutOfMemoryError):                # what the allocator has left over of earlier tests
            for _ in range(limit // (16 << 20) + 2):
                held.append(torch.empty(16 << 20, dtype=torch.uint8, device=DEV))
        torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + grad_bytes + (8 << 20)) / total)
        assert binding.grad_dense(g, ids1, ids2, None, n) is None
        room = torch.empty(grad_bytes, dtype=torch.uint8, device=DEV)   # the attempt holds nothing back
        del room
    finally:
        held.clear()
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert binding.grad_dense(g, ids1, ids2, None, n) is not None
