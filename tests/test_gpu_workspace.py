"""The workspace that the short form of beaver_matmul allocates where memory is short: what the call needs, without making the
allocator give its cache back first."""
import pytest
import torch

from paper_2402_02320_amd import spin

pytestmark = pytest.mark.gpu
DIMS = (2, 1, 2048, 2048, 2048)


def uniform(g, *shape):
    return torch.empty(shape, dtype=torch.int64, device="cuda").random_(-2 ** 63, 2 ** 63 - 1, generator=g)


def operands(n, batch, M, N, K):
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    return [uniform(g, n, batch, *s) for s in ((M, K), (K, N), (M, K), (K, N), (M, N))]


@pytest.fixture
def short_memory():
    """The process may take what its tensors, a call's result and the workspace it needs take, and little more."""
    torch.cuda.empty_cache()
    ops = operands(*DIMS)
    need, most = spin.beaver_matmul_workspace_bytes(*DIMS), spin.beaver_matmul_preferred_workspace_bytes(*DIMS)
    assert most > need + 3 * ops[4].nbytes + (128 << 20)
    total = torch.cuda.mem_get_info()[1]
    share = torch.cuda.get_per_process_memory_fraction()
    torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + 4 * ops[4].nbytes + need + (64 << 20)) / total)
    yield ops
    torch.cuda.set_per_process_memory_fraction(share)


def test_no_cache_flush_where_the_preferred_size_does_not_fit(short_memory):
    ops = short_memory
    flushes = torch.cuda.memory_stats()["num_alloc_retries"]
    got = [spin.beaver_matmul(*ops) for _ in range(3)]
    assert torch.cuda.memory_stats()["num_alloc_retries"] == flushes
    want = spin.beaver_matmul(*ops, workspace=torch.empty(spin.beaver_matmul_workspace_bytes(*DIMS), dtype=torch.uint8, device="cuda"))
    assert all(torch.equal(z, want) for z in got)


def test_the_preferred_size_where_it_fits():
    ops = operands(*DIMS)
    torch.cuda.synchronize()
    before = torch.cuda.memory_allocated()
    torch.cuda.reset_peak_memory_stats()
    spin.beaver_matmul(*ops, out=ops[4])
    assert torch.cuda.max_memory_allocated() - before >= spin.beaver_matmul_preferred_workspace_bytes(*DIMS)


def test_short_form_under_capture():
    ops = operands(*DIMS)
    want = spin.beaver_matmul(*ops)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        got = spin.beaver_matmul(*ops)
    for _ in range(3):
        got.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(got, want)
