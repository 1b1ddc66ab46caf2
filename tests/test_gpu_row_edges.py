"""The row kernel where its k-tiles, its 16-byte rows and its halved units have edges: odd inner dimensions (element-wise loads; the last
k-tile of one to 32), odd and even numbers of k-tiles (an odd one is padded by a tile without products), one to three parties (units whole
and in parts), one and two column halves, a workgroup with one item and with several; single and grouped, C in place.  The kernel is asked
for by name; that the row kernel made them shows in the workspace too, whose first part (left fragments) it leaves as it was.  Exact ring words."""
import pytest
import torch

from paper_2402_02320_amd import spin

pytestmark = pytest.mark.gpu

SHAPES = [(3, 1, 8192, 64, 31), (2, 64, 300, 64, 33), (3, 100, 128, 64, 63), (3, 20, 800, 65, 65), (2, 33, 260, 31, 95), (3, 1, 16385, 64, 97),
          (3, 9, 1000, 64, 127), (2, 1, 20000, 64, 129), (1, 64, 320, 64, 47), (1, 1, 33000, 40, 161), (3, 128, 64, 40, 225), (3, 255, 20, 1, 33)]


@pytest.mark.parametrize("n,batch,M,N,K", SHAPES)
@pytest.mark.parametrize("transposed", [False, True])
def test_words(n, batch, M, N, K, transposed):
    g = torch.Generator(device="cuda")
    g.manual_seed(M + K)

    def u(*s):
        return torch.empty(s, dtype=torch.int64, device="cuda").random_(-2 ** 63, 2 ** 63 - 1, generator=g)
    y = (N, K) if transposed else (K, N)
    X, Y, A, B, C = u(n, batch, M, K), u(n, batch, *y), u(n, batch, M, K), u(n, batch, *y), u(n, batch, M, N)
    want = spin.beaver_matmul(X, Y, A, B, C, path=spin.VALU, y_transposed=transposed)
    size = spin.beaver_matmul_workspace_bytes(n, batch, M, N, K)
    left = (n + 1) * batch * ((M + 127) // 128 * 4) * ((K + 31) // 32) * 8192
    ws = torch.full((2 * size,), 0x5A, dtype=torch.uint8, device="cuda")

    def rows(parts):                                     # the left part as it was, the right one written
        for at in range(0, parts * size, size):
            kept, packed = bool((ws[at:at + left] == 0x5A).all()), not bool((ws[at + left:at + size] == 0x5A).all())
            assert kept and packed, "not a product of the row kernel"
    assert torch.equal(spin.beaver_matmul_by("rows", 1, X, Y, A, B, C, y_transposed=transposed, workspace=ws), want)
    rows(1)
    group = dict(X=X, Y=Y, A=A, B=B, C=C, y_transposed=transposed)
    assert all(torch.equal(z, want) for z in spin.beaver_matmul_grouped_by("rows", [group, group], workspace=ws))
    rows(2)
    assert torch.equal(spin.beaver_matmul_by("rows", 1, X, Y, A, B, C, out=C, y_transposed=transposed, workspace=ws), want)
