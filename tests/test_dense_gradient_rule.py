"""Which calls the autograd function's table gradient takes row by row: the rule's lines (fsa_mean_bwd_dense_pays), from both
sides.  The library's host code answers; no GPU."""
import pytest
import torch


@pytest.fixture(scope="module")
def pays():
    from paper_2511_13645_amd import binding, build
    if build.is_stale():
        build.build_hip()
    return lambda B, k1, k2, D, dtype, n: binding.fsa_mean_bwd_dense_pays(B, k1, k2, D, dtype, n)


F32, BF16 = torch.float32, torch.bfloat16


def test_two_hops_on_a_table_that_the_batch_covers(pays):
    assert pays(1024, 25, 10, 128, F32, 169343) and pays(1024, 25, 10, 128, BF16, 169343)
    assert pays(65536, 25, 10, 128, F32, 169343) and pays(8192, 15, 10, 100, F32, 2449029)
    assert not pays(64, 25, 10, 128, F32, 169343)


@pytest.mark.parametrize("B,k,D,n", [(16384, 15, 128, 15000), (65536, 30, 16, 10000), (30000, 10, 64, 500000)])
def test_one_hop_is_left_to_the_atomics(pays, B, k, D, n):
    assert not pays(B, k, 0, D, F32, n)


@pytest.mark.parametrize("rows_per_slot,taken", [(0.5, True), (2, True), (2.5, False), (10, False)])
def test_tables_of_mostly_unnamed_rows_are_left_to_the_fill(pays, rows_per_slot, taken):
    assert pays(1024, 25, 10, 128, F32, int(256000 * rows_per_slot)) == taken


@pytest.mark.parametrize("B,k1,k2,D,n,taken", [
    (1024, 15, 10, 128, 300, False),                                    # nineteen bins
    (1024, 25, 10, 64, 2100, False),
    (1024, 25, 10, 64, 20000, True),
    (8192, 25, 10, 64, 20000, True),
    (65536, 25, 10, 64, 20000, False),                                  # 13,000 slots to a bin
    (8192, 15, 10, 32, 20000, False),                                   # rows of 128 bytes
    (65536, 30, 10, 16, 10000, False),
])
def test_small_tables_and_narrow_rows_are_left_to_the_atomics(pays, B, k1, k2, D, n, taken):
    assert pays(B, k1, k2, D, F32, n) == taken


@pytest.mark.parametrize("B,D,n,taken", [(555, 300, 30000, True), (555, 301, 30000, False), (1024, 602, 232965, True), (270, 602, 60000, False)])
def test_rows_that_are_not_made_of_quads_need_a_larger_call(pays, B, D, n, taken):
    assert pays(B, 25, 10, D, F32, n) == taken


@pytest.mark.parametrize("B,k1,k2,n", [(2 ** 60, 64, 64, 1000), (2 ** 62, 4, 0, 1000), (2 ** 63 - 1, 1, 1, 1), (16, 4, 4, 2 ** 31), (16, 4, 4, 2 ** 62)])
def test_no_workspace_for_sizes_that_the_call_refuses(pays, B, k1, k2, n):
    """Products of such sizes leave 64 bits; the call itself answers FSA_ERR_ARG."""
    from paper_2511_13645_amd import binding
    assert binding.fsa_mean_bwd_dense_workspace_bytes(B, k1, k2, 8, n) == 0
    assert not pays(B, k1, k2, 64, F32, n)
