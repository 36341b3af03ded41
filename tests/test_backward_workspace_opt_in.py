"""The Python backward calls hand the library the caller's workspace and nothing else: without one they
allocate nothing and the library adds with atomics, which calls on other streams and threads may do to the
same gradient table at the same time.  Runs on the CPU with a stand-in for the library that records what it
was called with."""
import pytest
import torch

from paper_2511_13645_amd import binding

B, K1, K2, K3, D, N = 1400, 10, 10, 2, 128, 50            # sizes at which the plain-store routes pay


class _Library:
    def __init__(self):
        self.calls = []

    def __getattr__(self, name):
        if name.endswith("_workspace_bytes"):
            return lambda *a: 4096
        return lambda *a: (self.calls.append((name, a)), 0)[1]


@pytest.fixture
def library(monkeypatch):
    L = _Library()
    monkeypatch.setattr(binding, "lib", lambda: L)
    monkeypatch.setattr(binding, "_need", lambda *a, **k: None)
    monkeypatch.setattr(binding, "_stream", lambda *a: 0)
    return L


def _calls():
    z = lambda *s: torch.zeros(s)
    i = lambda *s: torch.zeros(s, dtype=torch.int32)
    g, gx, i1, i2, i3 = z(B, D), z(N, D), i(B, K1), i(B, K1, K2), i(B, K1, K2, K3)
    return {
        "fsa_mean_bwd_ws": lambda **k: binding.fsa_mean_bwd_ws(g, i1, i2, grad_x=gx, **k),
        "fsa_mean_bwd_lp": lambda **k: binding.fsa_mean_bwd_lp(g, i1, i2, grad_x=gx, **k),
        "fsa_wmean_bwd": lambda **k: binding.fsa_wmean_bwd(g, i1, z(B, K1), i2, z(B, K1, K2), grad_x=gx, **k),
        "fsa_mean3_bwd": lambda **k: binding.fsa_mean3_bwd(g, i1, i2, i3, grad_x=gx, **k),
        "fsa_mean_bwd": lambda **k: binding.fsa_mean_bwd(g, i1, i2, grad_x=gx, **k),
    }


@pytest.mark.parametrize("name", ["fsa_mean_bwd", "fsa_mean_bwd_ws", "fsa_mean_bwd_lp", "fsa_wmean_bwd", "fsa_mean3_bwd"])
def test_no_workspace_unless_the_caller_brings_one(library, monkeypatch, name):
    call = _calls()[name]
    sizes, empty = [], torch.empty
    monkeypatch.setattr(torch, "empty", lambda *a, **k: (sizes.append(a[0]), empty(*a, **k))[1])
    call()
    assert sizes == ([(B, K1, D)] if name == "fsa_mean3_bwd" else []), "nothing but the three-hop call's `work`"
    entry, args = library.calls[-1]
    if entry.endswith("_ws"):
        assert args[-3] is None and args[-2] == 0, "no address and no bytes"
    else:
        assert entry == name


@pytest.mark.parametrize("name", ["fsa_mean_bwd_ws", "fsa_mean_bwd_lp", "fsa_wmean_bwd", "fsa_mean3_bwd"])
def test_the_callers_workspace_reaches_the_library(library, name):
    ws = torch.zeros(300, dtype=torch.int16)
    _calls()[name](workspace=ws)
    entry, args = library.calls[-1]
    assert entry == (name if name.endswith("_ws") else name + "_ws")
    assert args[-3] == ws.data_ptr() and args[-2] == 600
