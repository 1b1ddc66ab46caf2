"""The row kernel's items: row blocks in eight contiguous shares, column tiles fastest.  Block counts around multiples of 8 and of the
workgroups a launch has, one to three column tiles, one batch entry and several, against the vector-ALU path.  Exact ring words."""
import pytest
import torch

from paper_2402_02320_amd import spin

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,batch,M,N,K", [(3, 1, 3 * 32, 64, 2048), (3, 1, 8 * 32 + 1, 40, 2048), (2, 9, 33, 64, 1024), (3, 15, 31, 70, 512), (1, 17, 64, 128, 512),
                                           (3, 64, 128, 128, 64), (3, 65, 127, 129, 64), (2, 1, 257 * 32, 64, 96), (3, 513, 32, 64, 64), (3, 511, 20, 100, 66)])
@pytest.mark.parametrize("transposed", [False, True])
def test_words(n, batch, M, N, K, transposed):
    g = torch.Generator(device="cuda")
    g.manual_seed(M + K)

    def u(*s):
        return torch.empty(s, dtype=torch.int64, device="cuda").random_(-2 ** 63, 2 ** 63 - 1, generator=g)
    y = (N, K) if transposed else (K, N)
    X, Y, A, B, C = u(n, batch, M, K), u(n, batch, *y), u(n, batch, M, K), u(n, batch, *y), u(n, batch, M, N)
    want = spin.beaver_matmul(X, Y, A, B, C, path=spin.VALU, y_transposed=transposed)
    assert torch.equal(spin.beaver_matmul(X, Y, A, B, C, y_transposed=transposed), want)
    group = dict(X=X, Y=Y, A=A, B=B, C=C, y_transposed=transposed)
    assert all(torch.equal(z, want) for z in spin.beaver_matmul_grouped([group, group]))
