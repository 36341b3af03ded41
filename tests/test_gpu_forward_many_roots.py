"""Calls of so many seeds that the threads of one launch for all of them would be 2^32 or more, which a launch
cuts off without an error.  A seed's results depend on the seed alone, so a batch that repeats a list of seeds has
to return that list's results again and again; the list alone is an ordinary call."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
N = 1000
B = (1 << 26) + 3                                   # a wave per root


@pytest.fixture(scope="module")
def fsa():
    from paper_2511_13645_amd import binding
    binding.lib()
    return binding


@pytest.fixture(scope="module")
def graph():
    """Nodes of 0 .. 4 neighbors, one feature each."""
    gen = torch.Generator(device=DEV).manual_seed(3)
    deg = torch.arange(N, device=DEV) % 5
    indptr = torch.zeros(N + 1, dtype=torch.int32, device=DEV)
    indptr[1:] = deg.cumsum(0)
    n_edges = int(indptr[-1])
    return dict(indptr=indptr, indices=torch.randint(0, N, (n_edges,), generator=gen, device=DEV, dtype=torch.int32),
                w=torch.rand(n_edges, generator=gen, device=DEV) + 0.5, x=torch.randn((N, 1), generator=gen, device=DEV),
                few=torch.arange(N, device=DEV, dtype=torch.int32), many=torch.arange(B, device=DEV, dtype=torch.int32) % N)


def _repeats(many, few):
    """Whether `many` is `few` over and over, and what is left of it at the end."""
    whole = many.shape[0] // few.shape[0] * few.shape[0]
    same = (many[:whole].view(-1, *few.shape) == few).all()
    return bool(same) and torch.equal(many[whole:], few[:many.shape[0] - whole])


def _check(many, few):
    many, few = (many, few) if isinstance(many, (tuple, list)) else ((many,), (few,))
    for i, (m, f) in enumerate(zip(many, few)):
        assert (m is None) == (f is None)
        if f is not None:
            assert m.shape[0] == B and _repeats(m, f), "output %d" % i


def test_two_hops_and_their_replay(fsa, graph):
    args = lambda seeds: (graph["indptr"], graph["indices"], graph["x"], seeds, [1, 1], 9)
    many, few = fsa.fsa_sample_mean_fwd(*args(graph["many"])), fsa.fsa_sample_mean_fwd(*args(graph["few"]))
    _check(many, few)
    _check(fsa.fsa_mean_replay_fwd(graph["x"], many[2], many[3]), few[:2])


def test_two_hops_weighted(fsa, graph):
    args = lambda seeds: (graph["indptr"], graph["indices"], graph["w"], graph["x"], seeds, [1, 1], 9)
    many, few = fsa.fsa_sample_wmean_fwd(*args(graph["many"])), fsa.fsa_sample_wmean_fwd(*args(graph["few"]))
    _check(many, few)
    _check(fsa.fsa_wmean_replay_fwd(graph["x"], many[2], many[4], many[3], many[5]), few[:2])


def test_one_hop_of_a_wave_per_seed(fsa, graph):
    """More than 32 neighbors a seed: not several seeds per wave."""
    args = lambda seeds: (graph["indptr"], graph["indices"], graph["x"], seeds, [33], 9)
    _check(fsa.fsa_sample_mean_fwd(*args(graph["many"])), fsa.fsa_sample_mean_fwd(*args(graph["few"])))


def test_three_hops(fsa, graph):
    args = lambda seeds: (graph["indptr"], graph["indices"], graph["x"], seeds, [1, 1, 1], 9)
    many = fsa.fsa_sample_mean3_fwd(*args(graph["many"]), emit_h2=True)
    few = fsa.fsa_sample_mean3_fwd(*args(graph["few"]), emit_h2=True)
    _check(list(many.values()), list(few.values()))


def test_one_hop_backward(fsa):
    """16 seeds per wave: 2^30 seeds are 2^32 threads.  Every node is named equally often, with a gradient of one."""
    nodes, seeds = 1 << 16, (1 << 30) + (1 << 16)
    ids = (torch.arange(seeds, device=DEV, dtype=torch.int32) % nodes).view(seeds, 1)
    gx = torch.zeros((nodes, 1), device=DEV)
    fsa.fsa_mean_bwd(torch.ones((seeds, 1), device=DEV), ids, grad_x=gx)
    assert bool((gx == seeds // nodes).all())
