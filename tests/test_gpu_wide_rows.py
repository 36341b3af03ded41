"""Gathers of rows wider than one tile: every number of tiles on each side of the kernels' sizes, pieces of 16, 8,
4 and 2 bytes, lists shorter than, equal to and longer than the rows in flight, weighted and not."""
import numpy as np
import pytest
import torch

from parity_util import TOL, assert_close, forward_scales, host_x, to_f64
from test_gpu_parity import fsa, ragged_graph, run_case  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D, bf16", [(640, False), (768, False), (772, False), (1280, False), (1284, False),     # 16-byte pieces
                                     (130, False), (386, False), (514, False), (642, False), (770, False), (962, False),  # 8
                                     (129, False), (193, False), (321, False), (511, False),                     # 4
                                     (1544, True), (772, True), (386, True), (129, True), (385, True)])          # 16, 8, 4, 2, 2
def test_tiles_and_pieces(fsa, orc, D, bf16):  # noqa: F811
    n = 500
    indptr, indices = ragged_graph(n, seed=D, max_deg=9, hub_deg=200)
    rng = np.random.default_rng(D)
    x = torch.from_numpy(rng.standard_normal((n, D)).astype(np.float32))
    x = x.to(torch.bfloat16) if bf16 else x
    seeds = np.concatenate([np.arange(8), rng.integers(0, n, 30)]).astype(np.int32)
    for fan in ([1], [2], [5], [9], [2, 1], [5, 3]):
        run_case(fsa, orc, indptr, indices, x, seeds, fan, 3, check_bwd=False, what="D=%d fan=%s" % (D, fan))
    run_case(fsa, orc, indptr, indices, x, np.resize(seeds, 4200), [3, 2], 3, check_bwd=False, what="one wave per root D=%d" % D)
    w = rng.random(indices.shape[0]).astype(np.float32) + 0.25
    up = lambda a: torch.from_numpy(a).to("cuda:0")
    hx, is_bf16 = host_x(x)
    for many, fan in ((seeds, [5, 3]), (np.resize(seeds, 4200), [3, 2])):
        ref = orc.sample_wmean_fwd(indptr, indices, w, hx, many, fan, 3, bf16=is_bf16)
        got = fsa.fsa_sample_wmean_fwd(up(indptr), up(indices), up(w), x.to("cuda:0"), up(many), fan, 3)
        torch.cuda.synchronize()
        a_out, a_h1 = forward_scales(x.to("cuda:0"), got[2], got[3])
        # weights from 0.25 to 1.25: a weighted mean of magnitudes is within five plain ones
        assert_close(to_f64(got[0]), ref[0], 5 * a_out, TOL[x.dtype], "weighted out")
        assert_close(to_f64(got[1]), ref[1], 5 * a_h1, TOL[x.dtype], "weighted out_h1")
