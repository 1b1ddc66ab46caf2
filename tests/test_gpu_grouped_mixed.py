"""A grouped Beaver matmul of products of different shapes, odd and even inner dimensions, as the library chooses: all by the row kernel or all
by half tiles, up to three parties, and by half tiles beyond.  Compared with the VALU path, and with more groups than one shared launch
holds.  (Each kernel by its name: test_gpu_named_kernels.py.)"""
import pytest
import torch

from paper_2402_02320_amd import spin

pytestmark = pytest.mark.gpu


def uniform(g, *shape):
    return torch.empty(shape, dtype=torch.int64, device="cuda").random_(-2 ** 63, 2 ** 63 - 1, generator=g)


@pytest.mark.parametrize("n", [1, 2, 3, 4])
@pytest.mark.parametrize("count", [2, 6, 36])
def test_groups_of_different_shapes(n, count):
    g = torch.Generator(device="cuda")
    g.manual_seed(n * 100 + count)
    shapes = [(2, 196, 96, 64, True), (3, 49, 32, 49, False), (1, 33, 64, 130, False), (2, 70, 65, 33, True), (1, 1, 1, 2, False),
              (1, 5, 7, 1, True)]
    groups = []
    for i in range(count):
        batch, M, N, K, tr = shapes[i % len(shapes)]
        y = (N, K) if tr else (K, N)
        groups.append(dict(X=uniform(g, n, batch, M, K), Y=uniform(g, n, batch, *y), A=uniform(g, n, batch, M, K),
                           B=uniform(g, n, batch, *y), C=uniform(g, n, batch, M, N), y_transposed=tr))
    way = spin.matmul_grouped_way(n, [shapes[i % len(shapes)] for i in range(count)])
    assert way in (("rows", "half") if n <= 3 else ("half",))
    want = spin.beaver_matmul_grouped(groups, path=spin.VALU)
    for _ in range(2):
        got = spin.beaver_matmul_grouped(groups)
        assert all(torch.equal(a, b) for a, b in zip(got, want))


# eight parties: few and many right-hand pack workgroups (the kernel of all packs has one wave a SIMD); with and without packs by rows
@pytest.mark.parametrize("shapes", [[(1, 64, 2048, 512, False), (2, 33, 65, 64, True)], [(1, 64, 2112, 512, False), (2, 33, 65, 64, True)],
                                    [(3, 20, 4100, 301, False)] * 3 + [(1, 70, 50, 33, True)], [(1, 64, 4096, 1000, False)]])
def test_eight_parties_many_right_operands(shapes):
    g = torch.Generator(device="cuda")
    g.manual_seed(len(shapes))
    groups = []
    for batch, M, N, K, tr in shapes:
        y = (N, K) if tr else (K, N)
        groups.append(dict(X=uniform(g, 8, batch, M, K), Y=uniform(g, 8, batch, *y), A=uniform(g, 8, batch, M, K),
                           B=uniform(g, 8, batch, *y), C=uniform(g, 8, batch, M, N), y_transposed=tr))
    want = spin.beaver_matmul_grouped(groups, path=spin.VALU)
    assert all(torch.equal(a, b) for a, b in zip(spin.beaver_matmul_grouped(groups), want))
