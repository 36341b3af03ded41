"""The backward that gives every destination row one owner (hashed buckets, one plain update per
row; calls that are handed a workspace) against the oracle, at sizes large enough to take it: every piece width and element type,
rows shared inside a tile, rows sampled too often for an owner, weights, three hops, a captured
graph.  Tolerances are those of the files that these calls are taken from: 1e-5 of the sum of the
contributions' magnitudes for fp32 tables, one rounding per addition for 16-bit ones."""
import numpy as np
import pytest
import torch

from parity_util import assert_close, marked_workspace, to_f64, workspace_route
from test_gpu_backward_workspace import _ids
from test_gpu_lowprec import COMBOS, lowprec_case
from test_gpu_parity import ragged_graph
from test_gpu_three_hop import three_hop_case
from test_gpu_weighted import _graph, _run

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def fsa():
    from paper_2511_13645_amd import binding
    binding.lib()
    return binding


def _workspace(fsa, B, k1, k2, D, dtype=torch.float32):
    need = fsa.fsa_bwd_workspace_bytes(B, k1, k2, D, dtype)
    assert need > 0
    return marked_workspace(need)


# pieces of 4 / 2 / 1 floats (D % 4, % 2, odd), one tile of lanes and more, several roots per tile and
# roots of more leaf slots than a tile, a last wave with few leaf slots, 16 and (from 288,000 leaf slots on) 32
# leaf slots per wave.  Rows of 1 KB and more in up to 512 pieces belong to the sorted route.
@pytest.mark.parametrize("B,k1,k2,D", [(1301, 10, 10, 100), (1301, 10, 10, 101), (701, 13, 9, 202), (90, 40, 30, 128),
                                       (37, 64, 64, 248), (25001, 1, 5, 128), (601, 10, 10, 1030), (8001, 5, 3, 515), (3001, 10, 10, 98)])
@pytest.mark.parametrize("with_h1", [False, True])
def test_every_row_has_one_owner(fsa, orc, B, k1, k2, D, with_h1):
    ws = _workspace(fsa, B, k1, k2, D)
    rng = np.random.default_rng(D + B)
    n = 30000 if B * k1 * k2 < 200000 else 100000                  # no row more than 16 times
    ids1, ids2 = _ids(rng, B, k1, k2, n)
    g = rng.standard_normal((B, D)).astype(np.float32)
    gh = rng.standard_normal((B, k1, D)).astype(np.float32) if with_h1 else None
    d = [None if a is None else torch.from_numpy(a).to(DEV) for a in (g, ids1, ids2, gh)]
    got = []
    for _ in range(2):
        gx = torch.full((n, D), 0.5, device=DEV)
        fsa.fsa_mean_bwd_lp(*d, grad_x=gx, workspace=ws)
        got.append(gx)
    torch.cuda.synchronize()
    assert workspace_route(ws) == "owned"
    ref = orc.mean_bwd(g.astype(np.float64), ids1, ids2, None if gh is None else gh.astype(np.float64), num_nodes=n)
    mag = orc.mean_bwd(np.abs(g).astype(np.float64), ids1, ids2, None if gh is None else np.abs(gh).astype(np.float64), num_nodes=n)
    assert_close(to_f64(got[0]) - 0.5, ref, mag + 0.5, 1e-5, "grad_x")
    assert torch.equal(got[0], got[1]), "no row is sampled more than 16 times: the result is reproducible"


@pytest.mark.parametrize("targets", [3, 300, 4000])
def test_rows_sampled_too_often_for_an_owner(fsa, orc, targets):
    """Three rows take everything; 300 rows overflow their buckets; 4000 rows are sampled about 35 times each."""
    rng = np.random.default_rng(targets)
    B, k1, k2, D, n = 1500, 10, 10, 104, 5000
    ids1, ids2 = _ids(rng, B, k1, k2, n, targets=rng.permutation(n)[:targets].astype(np.int32))
    ws = _workspace(fsa, B, k1, k2, D)
    g = rng.standard_normal((B, D)).astype(np.float32)
    gx = torch.zeros((n, D), device=DEV)
    fsa.fsa_mean_bwd_lp(torch.from_numpy(g).to(DEV), torch.from_numpy(ids1).to(DEV), torch.from_numpy(ids2).to(DEV), grad_x=gx,
                        workspace=ws)
    torch.cuda.synchronize()
    assert workspace_route(ws) == "owned"
    ref = orc.mean_bwd(g.astype(np.float64), ids1, ids2, num_nodes=n)
    mag = orc.mean_bwd(np.abs(g).astype(np.float64), ids1, ids2, num_nodes=n)
    assert_close(to_f64(gx), ref, mag, 1e-5, "grad_x")


@pytest.mark.parametrize("g_dtype,x_dtype", COMBOS)
@pytest.mark.parametrize("D", [248, 202])
def test_element_types(fsa, orc, g_dtype, x_dtype, D):
    n, fan, B = 20000, [15, 10], 930
    ws = _workspace(fsa, B, *fan, D, x_dtype)
    indptr, indices = ragged_graph(n, seed=D)
    seeds = np.concatenate([np.arange(8), np.random.default_rng(D).integers(0, n, B - 8)]).astype(np.int32)
    lowprec_case(fsa, orc, indptr, indices, n, D, seeds, fan, g_dtype, x_dtype, "%s -> %s" % (g_dtype, x_dtype),
                 workspace=ws)
    assert workspace_route(ws) == "owned"


@pytest.mark.parametrize("D", [100, 257])
def test_weighted(fsa, orc, D):
    n, fan, B = 20000, [15, 10], 1000
    ws = _workspace(fsa, B, *fan, D)
    indptr, indices, ew = _graph(n, seed=D)
    rng = np.random.default_rng(D)
    x = torch.from_numpy(rng.standard_normal((n, D)).astype(np.float32))
    seeds = np.concatenate([np.arange(24), rng.integers(0, n, B - 24)]).astype(np.int32)
    _run(fsa, orc, indptr, indices, ew, x, seeds, fan, 7, "weighted D=%d" % D, workspace=ws)
    assert workspace_route(ws) == "owned"


def test_three_hops(fsa, orc):
    n, fan, B, D = 20000, [9, 8, 7], 260, 128
    ws = _workspace(fsa, B * fan[0], fan[1], fan[2], D)
    indptr, indices = ragged_graph(n, seed=2, max_deg=30)
    rng = np.random.default_rng(4)
    x = torch.from_numpy(rng.standard_normal((n, D)).astype(np.float32))
    three_hop_case(fsa, orc, indptr, indices, x, np.arange(B).astype(np.int32), fan, 9, "three hops", workspace=ws)
    assert workspace_route(ws) == "owned"


def test_captured_graph(fsa):
    rng = np.random.default_rng(6)
    B, k1, k2, D, n = 1400, 10, 10, 100, 200000
    ws = _workspace(fsa, B, k1, k2, D)
    ids1, ids2 = (torch.from_numpy(a).to(DEV) for a in _ids(rng, B, k1, k2, n))
    g, gx = torch.randn((B, D), device=DEV), torch.zeros((n, D), device=DEV)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        fsa.fsa_mean_bwd_lp(g, ids1, ids2, grad_x=gx, workspace=ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        gx.zero_()
        fsa.fsa_mean_bwd_lp(g, ids1, ids2, grad_x=gx, workspace=ws)
    for turn in range(4):
        g.normal_()                                                  # eager work between the replays
        graph.replay()
        torch.cuda.synchronize()
        want = torch.zeros_like(gx)
        fsa.fsa_mean_bwd_lp(g, ids1, ids2, grad_x=want, workspace=ws)
        torch.cuda.synchronize()
        assert torch.equal(gx, want), turn
