"""The binding's native host path against its Python path: the same outputs bit for bit, the same errors, and
calls that are not plain left to the Python path."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fsa():
    from paper_2511_13645_amd import binding
    binding.lib()
    return binding


@pytest.fixture(scope="module")
def data():
    rng = np.random.default_rng(0)
    n = 3000
    deg = rng.integers(0, 40, n)
    up = lambda a: torch.from_numpy(a).to("cuda:0")
    indptr = up(np.concatenate([[0], np.cumsum(deg)]).astype(np.int32))
    indices = up(rng.integers(0, n, int(deg.sum())).astype(np.int32))
    return dict(indptr=indptr, indices=indices, w=torch.rand(indices.shape[0], device="cuda:0"), n=n,
                seeds=up(rng.integers(0, n, 77).astype(np.int32)))


class _Counting:
    """Stands in for _fsa_host and notes which calls it took."""
    def __init__(self, host):
        self.host, self.took = host, []

    def __getattr__(self, name):
        def call(*a):
            r = getattr(self.host, name)(*a)
            self.took.append(r is not None)
            return r
        return call


def _calls(fsa, d, x, fan):
    """Every entry point with a native path: name -> outputs."""
    D, gx = x.shape[1], torch.zeros(x.shape, device=x.device)
    r = {}
    for ids in (True, False):
        r["fwd %s" % ids] = fsa.fsa_sample_mean_fwd(d["indptr"], d["indices"], x, d["seeds"], fan, 5, emit_ids=ids, emit_h1=ids)
        r["wfwd %s" % ids] = fsa.fsa_sample_wmean_fwd(d["indptr"], d["indices"], d["w"], x, d["seeds"], fan, 5, emit_ids=ids, emit_h1=ids)
    i1, i2, w1, w2 = r["wfwd True"][2:]
    r["replay"] = fsa.fsa_mean_replay_fwd(x, i1, i2)
    one = torch.ones((len(d["seeds"]), D), device=x.device)      # one seed at a time per row: no order to differ in
    one[1:] = 0
    r["bwd"] = fsa.fsa_mean_bwd(one, i1, i2, grad_x=gx.clone())
    r["bwd_ws"] = fsa.fsa_mean_bwd_ws(one, i1, i2, grad_x=gx.clone())
    r["bwd_lp"] = fsa.fsa_mean_bwd_lp(one.to(x.dtype), i1, i2, grad_x=gx.clone())
    r["wbwd"] = fsa.fsa_wmean_bwd(one, i1, w1, i2, w2, grad_x=gx.clone())
    return r


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.float16])
@pytest.mark.parametrize("fan", [[6], (7, 4)])
def test_same_results_as_the_python_path(fsa, data, monkeypatch, fan, dtype):
    x = torch.nn.Parameter(torch.randn((data["n"], 36), device="cuda:0").to(dtype))
    count = _Counting(fsa._host)
    monkeypatch.setattr(fsa, "_host", count)
    with torch.no_grad():
        native = _calls(fsa, data, x, fan)
        assert len(count.took) == 9 and all(count.took)
        monkeypatch.setattr(fsa, "_host", None)
        python = _calls(fsa, data, x, fan)
    for name, want in python.items():
        got = native[name]
        want, got = (want, got) if isinstance(want, tuple) else ((want,), (got,))
        assert len(got) == len(want)
        for a, b in zip(got, want):
            assert (a is None) == (b is None), name
            if a is not None:
                assert a.dtype == b.dtype and a.shape == b.shape and type(a) is type(b) and a.requires_grad == b.requires_grad, name
                if "bwd" in name:                  # a root's slots may share a row: two or three additions in either order
                    assert torch.allclose(a, b, rtol=1e-6, atol=1e-7), name
                else:
                    assert torch.equal(a, b), name


def test_what_is_not_plain_is_left_to_the_python_path(fsa, data, monkeypatch):
    x = torch.randn((data["n"], 36), device="cuda:0")
    count = _Counting(fsa._host)
    monkeypatch.setattr(fsa, "_host", count)
    p, i, s = data["indptr"], data["indices"], data["seeds"]
    want = fsa.fsa_sample_mean_fwd(p, i, x, s, [6, 3], 5)
    assert count.took.pop() is True
    same = lambda got: all(torch.equal(a, b) for a, b in zip(got, want))
    assert same(fsa.fsa_sample_mean_fwd(p, i, x, s, (np.int64(6), 3), 5)) and count.took.pop() is False
    with torch.device("cuda:0"):                   # a function mode
        assert same(fsa.fsa_sample_mean_fwd(p, i, x, s, [6, 3], 5)) and count.took.pop() is False
    n_took = len(count.took)
    assert same(fsa.fsa_sample_mean_fwd(p, i, x, s, [6, 3], 5, stream=torch.cuda.current_stream()))
    assert same(fsa.fsa_sample_mean_fwd(p, i, x, s, [6, 3], 5, out=torch.empty((77, 36), device="cuda:0")))
    assert len(count.took) == n_took
    for bad, error in ((dict(x=x.t()), ValueError), (dict(s=s.long()), TypeError), (dict(x=x.double()), TypeError),
                       (dict(p=p[:-1]), ValueError), (dict(s=s.cpu()), ValueError), (dict(fan=[0, 3]), fsa.FsaError),
                       (dict(fan=[65]), fsa.FsaError)):
        a = dict(p=p, i=i, x=x, s=s, fan=[6, 3])
        a.update(bad)
        with pytest.raises(error):
            fsa.fsa_sample_mean_fwd(a["p"], a["i"], a["x"], a["s"], a["fan"], 5)
        assert count.took.pop() is False
    odd = torch.zeros((data["n"], 35), dtype=torch.bfloat16, device="cuda:0")
    with pytest.raises(fsa.FsaError):              # refused by the library: the native path's status, the same exception
        fsa.fsa_mean_bwd_lp(torch.zeros((77, 35), device="cuda:0"), want[2], want[3], grad_x=odd)
    assert count.took.pop() is True


def test_replay_and_backward_refuse_what_the_python_path_refuses(fsa, data, monkeypatch):
    """One argument wrong at a time: the native path leaves the call alone, and the caller sees the error that the
    binding raises without it."""
    x = torch.randn((data["n"], 36), device="cuda:0")
    _, _, i1, i2, w1, w2 = fsa.fsa_sample_wmean_fwd(data["indptr"], data["indices"], data["w"], x, data["seeds"], [6, 3], 5)
    B = len(data["seeds"])
    count = _Counting(fsa._host)

    def refused(call, **good):
        wrong = {"dtype": lambda t: t.double(), "host": lambda t: t.cpu(), "strides": lambda t: t.transpose(0, -1),
                 "batch": lambda t: t[1:].contiguous(), "width": lambda t: t[..., 1:].contiguous(), "dims": lambda t: t[None]}
        for name, t in good.items():
            for how, bad in wrong.items():
                if how == "width" and name in ("x", "ids2") and call == fsa.fsa_mean_replay_fwd or (name, how) == ("ids2", "width") and "w2" not in good:
                    continue                       # another width, other fanouts: a call of its own
                if name in ("x", "grad_x") and how == "batch":
                    continue                       # a smaller table is a table
                args = dict(good, **{name: bad(t)})
                seen = []
                for host in (count, None):
                    monkeypatch.setattr(fsa, "_host", host)
                    with pytest.raises(Exception) as e:
                        call(**args)
                    seen.append((e.type, str(e.value)))
                assert count.took.pop() is False and seen[0] == seen[1], (call.__name__, name, how)

    refused(fsa.fsa_mean_replay_fwd, x=x, ids1=i1, ids2=i2)
    g, gh, gx = torch.zeros((B, 36), device="cuda:0"), torch.zeros((B, 6, 36), device="cuda:0"), torch.zeros_like(x)
    for call in (fsa.fsa_mean_bwd, fsa.fsa_mean_bwd_ws, fsa.fsa_mean_bwd_lp):
        refused(call, grad_out=g, ids1=i1, ids2=i2, grad_h1=gh, grad_x=gx)
    refused(fsa.fsa_wmean_bwd, grad_out=g, ids1=i1, w1=w1, ids2=i2, w2=w2, grad_h1=gh, grad_x=gx)
    assert not count.took
