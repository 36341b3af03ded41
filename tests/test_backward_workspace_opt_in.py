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


@pytest.mark.parametrize("b,k1,k2,d,slot_rows", [(1200, 15, 10, 300, False), (256, 15, 10, 256, False),       # wide, under 32 MiB of them
                                                 (1024, 25, 10, 602, True), (4096, 15, 10, 100, True)])
def test_room_for_slot_rows_only_where_a_call_writes_them(b, k1, k2, d, slot_rows):
    leaves, up = b * k1 * k2, lambda v: (v + 255) // 256 * 256
    buckets = 1
    while buckets * (32 if d * 4 >= 1024 else 64) < leaves:
        buckets *= 2
    need = up(buckets * 128) + 256 + up(b * k1 * 8) + up(buckets * 256 * 8) + up(leaves * 8)
    if slot_rows:
        need += up(b * k1 * d * 4)
    assert binding.fsa_mean_bwd_workspace_bytes(b, k1, k2, d) == need


def test_calls_of_more_roots_than_a_launch_takes_have_no_sorted_route():
    assert binding.fsa_mean_bwd_workspace_bytes((1 << 24) - 1, 1, 1, 64) > 0
    assert binding.fsa_mean_bwd_workspace_bytes(1 << 24, 1, 1, 64) == 0
